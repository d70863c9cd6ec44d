// Several time steps per launch on tiles that fit into the LDS of one block.
//
// A block loads the post-collision populations of a tile of nodes and a halo
// of `halo` nodes around it, takes up to `halo` steps there and stores the
// tile.  Each step makes one more node of the halo stale, so the nodes a step
// computes shrink from the loaded region to the tile; a direction in which the
// region covers the whole period has no halo and wraps inside the block.
// Blocks never wait for each other: halo nodes are computed by every block
// that needs them, from the same values and with the same code, so the
// results do not depend on the tiling or on how a run is split over launches.
//
// A single step is bound by memory traffic on large plane domains and by the
// length of a launch on small ones (4 us for a few hundred nodes); both are
// shared by the steps of a launch here.  What remains is the issue rate of the
// collisions and the load of the region (large domains: two blocks per CU, one
// loads while the other computes) or a chain of LDS and arithmetic latencies
// with three barriers, 0.6 to 0.9 us per step (small ones).  Single steps and
// tiles, us per step: D2Q9 FP64 64x64 4.7 and 1.3, 1024x512 16.7 and 7.4,
// 1999x1501 71 and 34; FP32 2048x2048 50.2 and 25.2; D3Q15 FP64 2x44x44 5.9
// and 2.0; 16^3 D3Q19 FP64 6.2 and 3.9.  On three-dimensional domains beyond
// some 24^3 that are not thin the halo costs more than it saves: 48^3 D3Q19 FP32
// 8.5 in single steps, 8.8 in tiles of 6^3 and two steps.
//
// In the LDS array a cut link (x_f, i) keeps its value f_i(x_f, t) in the slot
// of direction i at its solid node x_f - e_i, which is where the pull of f_i
// at x_f reads and which no fluid node writes; so the pull needs no lookup.
#include <algorithm>

#include "engine.hpp"
#include "kernels.hpp"
#include "params.hpp"

namespace lbe {

constexpr int kTileThreads = 512;

// Nodes a region may have, by the bytes of a node's populations (all but the
// one at rest, which stays in its thread's registers): the LDS of a CU
// (160 KiB) holds two blocks.
template <class L, class T>
struct TileShape {
    static constexpr int NT = kTileThreads;
    static constexpr int NPT = L::Q * sizeof(T) <= 40 ? 4 : L::Q * sizeof(T) <= 76 ? 2 : 1;
    static constexpr int CAP = NT * NPT;                             // nodes of a region
    // links of a region: one of each thread, and as many whose f_i and f_ibar
    // wait in LDS instead of registers
    static constexpr int LINKS = 2 * NT;
    static constexpr size_t LDS = ((size_t)CAP * (L::Q - 1) + 2 * NT) * sizeof(T);
    static_assert((L::Q - 1) * CAP <= 65536 && 2 * LDS <= 160 * 1024, "region limits");
    // waves per SIMD the registers are shared by: two blocks of a CU, or one
    // where the populations of a node alone would overflow half a share
    static constexpr int WAVES = L::Q * sizeof(T) > 100 ? 2 : 4;
};

struct TileArgs {
    const uint32_t* first;      // links of the regions (TileLinks)
    const uint4* link;
    uint32_t blocks, per_xcd, ntile[2];
    int tile[3], region[3];
    uint32_t by_x, by_xy;       // ceil(2^22 / region row), / region plane
    int halo;
    uint32_t wrap;      // bit a: the region covers the period of direction a
    int steps;          // 1 .. halo
    // drag of the steps s with s0 <= s < s1 (TileDrag)
    double* acc;
    const int32_t* lktag;
    int tag, s0, s1;
    double weight;
    double ws[kTileSteps];   // factor on the wall terms of each step
};

// the outputs of each step (null: not stored); the last step's are always given
template <class T>
struct TileOut {
    T* f[kTileSteps];
    T* wa[kTileSteps];
};

// What a thread keeps of a region node: bits 1..18 the cut-link directions,
// 19..23 how many nodes it is away from the region's edge (31: no edge), 24 a
// node of the tile itself, 25..30 at the low and high end of x, y and z (x: of
// the domain; y, z: of the region), 31 solid or absent.
constexpr int kStEdge = 19, kStMine = 24, kStEnd = 25;
// whether a step that leaves `need` stale layers computes the node
__device__ __forceinline__ bool st_live(uint32_t st, int need) {
    return !is_solid(st) && (int)((st >> kStEdge) & 31u) >= need;
}
// a value the compiler cannot derive other values from ahead of their use:
// what is computed from it stays inside the step loop instead of in registers
// held across it
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}

// WRAP: some direction of the region wraps; without it the neighbours lie at
// offsets that are the same for every node.
template <class L, class T, int XB, bool WRAP>
__global__ void __launch_bounds__(kTileThreads, (TileShape<L, T>::WAVES))
k_tile_steps(const T* __restrict__ A, const T* __restrict__ waA, TileOut<T> out, NodeMeta nm,
             const LinkCoefT<T>* __restrict__ lkcoef, Grid g, Params<L, T> p, TileArgs a) {
    using S = TileShape<L, T>;
    constexpr int Q = L::Q, NT = S::NT, NPT = S::NPT, CAP = S::CAP;
    extern __shared__ char smem[];
    T* __restrict__ F = (T*)smem;                                    // F[(i - 1) * CAP + r]
    T* __restrict__ later = F + (Q - 1) * CAP;                       // of links past the NT-th
    // what each step needs of the arguments: a first read of each of their
    // cache lines inside the step loop would cost a memory round trip
    __shared__ T* out_f[kTileSteps];
    __shared__ T* out_wa[kTileSteps];
    __shared__ double wall_scale[kTileSteps];
    const int t = threadIdx.x;
    if (t < kTileSteps) {
        out_f[t] = out.f[t];
        out_wa[t] = out.wa[t];
        wall_scale[t] = a.ws[t];
    }
    const int RX = a.region[0], RY = a.region[1], RZ = a.region[2], RXY = RX * RY, R = RXY * RZ;

    // ---- load: the links this thread carries, its nodes' words and populations
    // The hardware deals blocks to the eight XCDs in turn; each takes the tiles
    // of one stretch, so that neighbours' halos are met in its own L2
    // (1999x1501 FP64 5% and 1024x512 8% less time per step).
    const uint32_t block = (blockIdx.x & 7u) * a.per_xcd + (blockIdx.x >> 3);
    if (block >= a.blocks) return;
    const uint32_t l0 = a.first[block], n_links = a.first[block + 1] - l0;
    const bool has_link = (uint32_t)t < n_links, has_more = (uint32_t)(t + NT) < n_links;
    const uint4 lk = has_link ? a.link[l0 + (uint32_t)t] : uint4{0u, 0u, 0u, 0u};
    uint32_t st[NPT], n[NPT];
    T f[NPT][Q];
    {
        const uint32_t yz = block / a.ntile[0];
        const int at[3] = {(int)(block - yz * a.ntile[0]), (int)(yz % a.ntile[1]),
                           (int)(yz / a.ntile[1])};
        const int dom[3] = {(int)g.nx, (int)g.ny, (int)g.nz};
#pragma unroll
        for (int m = 0; m < NPT; ++m) {
            const int r = t + m * NT;
            st[m] = kInfoSolid;
            n[m] = 0u;
            unroll<Q>([&](auto I) { f[m][decltype(I)::value] = T(0); });
            if (r >= R) continue;
            // r < 2^11: the quotients are exact
            const int z = (int)(((uint64_t)(uint32_t)r * a.by_xy) >> 22), rz = r - z * RXY;
            const int y = (int)(((uint64_t)(uint32_t)rz * a.by_x) >> 22);
            const int loc[3] = {rz - y * RX, y, z};
            int gl[3], edge = 31;
            bool mine = true;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const bool wrap = (a.wrap >> c) & 1u;
                const int u = at[c] * a.tile[c] - (wrap ? 0 : a.halo) + loc[c];
                if (!wrap) {
                    edge = min(edge, min(loc[c], a.region[c] - 1 - loc[c]));
                    mine = mine && loc[c] >= a.halo && loc[c] < a.halo + a.tile[c] && u < dom[c];
                }
                gl[c] = u < 0 ? u + dom[c] : u >= dom[c] ? u - dom[c] : u;
            }
            n[m] = (uint32_t)gl[0] + g.nx * ((uint32_t)gl[1] + g.ny * (uint32_t)gl[2]);
            const uint32_t info = nm.info[n[m]];
            unroll<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                f[m][i] = ldp<Q>(A, i, n[m]);
            });
            st[m] = (info & (kInfoSolid | kInfoMask)) | (uint32_t)edge << kStEdge |
                    (uint32_t)mine << kStMine | (uint32_t)(gl[0] == 0) << kStEnd |
                    (uint32_t)(gl[0] + 1 == dom[0]) << (kStEnd + 1) |
                    (uint32_t)(loc[1] == 0) << (kStEnd + 2) |
                    (uint32_t)(loc[1] + 1 == RY) << (kStEnd + 3) |
                    (uint32_t)(loc[2] == 0) << (kStEnd + 4) |
                    (uint32_t)(loc[2] + 1 == RZ) << (kStEnd + 5);
        }
    }
    T slot = has_link ? waA[lk.y] : T(0);
    // Whether the link counts in the drag of these steps, and its sum so far;
    // the own link of a thread is summed in registers: a read and a write of
    // its sum in every step stand in the chain of the steps (1024x512 FP64, 200
    // steps with drag and a read of the fields 2458 -> 2350 us).
    auto drags = [&](const uint4& l) {
        return a.acc && ((l.x >> 5) & 1u) && ((l.x >> 7) & 3u) != 1u && a.lktag[l.y] == a.tag;
    };
    // its weight, -e_ix times the window's: without a condition of the link's own
    // left, the drag is one branch of the launch in a step (80x42 FP64 without
    // drag 636 -> 632 us)
    auto weight_of = [&](const uint4& l) { return a.weight * (1.0 - (double)((l.x >> 7) & 3u)); };
    bool drag_own = false;
    double drag = 0.0, drag_weight = 0.0;
    unsigned long long counted = 0ull;   // by one thread: the steps before these
    if (a.acc) {
        drag_own = has_link && drags(lk);
        if (drag_own) {
            drag_weight = weight_of(lk);
            drag = a.acc[lk.y];
        }
        if (block == 0 && t == 0) counted = *step_count(a.acc);
    }
#pragma unroll
    for (int m = 0; m < NPT; ++m)
        if (!is_solid(st[m]))
            unroll<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                if constexpr (i > 0) F[(i - 1) * CAP + t + m * NT] = f[m][i];
            });
    // a link's f_ibar as pulled at its node, seam term included
    auto pulled_ibar = [&](const uint4& l) {
        T v = F[l.z >> 16];
        if constexpr (XB == XBC_PRESSURE) {
            const int sign = (int)((l.x >> 9) & 3u) - 1;
            if (sign != 0) {
                const bool axis = (l.x >> 6) & 1u;
                if constexpr (kStepTables<T>) {
                    const T w = axis ? p.seam[1] : p.seam[Q - 1];
                    v = sign > 0 ? v + w : v - w;
                } else {
                    v = fma(T(sign) * T(axis ? L::W[1] : L::W[Q - 1]), p.drho, v);
                }
            }
        }
        return v;
    };
    __syncthreads();
    // a link's slot: with Eq. (211) the stored value is completed with
    // c1 f_ibar(x_f, t)
    auto fill_slot = [&](const uint4& l, T v) {
        if (p.c1d) {
            const double c = p.c1d[l.y];
            if (c != 0.0) v = (T)((double)v + c * (double)pulled_ibar(l));
        }
        F[l.z & 0xFFFFu] = v;
    };
    if (has_link) fill_slot(lk, slot);
    if (has_more) {
        const uint4 l = a.link[l0 + (uint32_t)(t + NT)];
        fill_slot(l, waA[l.y]);
    }
    // all loads are back here; said outright, because else the compiler waits
    // for f in every step, and so for the coefficients each step loads ahead
    __builtin_amdgcn_s_waitcnt(0);
    if (a.acc)
        if (block == 0 && t == 0)
            *step_count(a.acc) = counted + (unsigned long long)(a.s1 - a.s0);
    __syncthreads();

    for (int s = 0; s < a.steps; ++s) {
        // nodes that are still correct after this step
        const int need = a.halo - a.steps + s + 1;
        // ---- pull
#pragma unroll
        for (int m = 0; m < NPT; ++m) {
            if (!st_live(st[m], need)) continue;
            const uint32_t word = opaque(st[m]);
            int x[3] = {1, 0, -1}, y[3] = {RX, 0, -RX}, z[3] = {RXY, 0, -RXY};   // of x - e: [e + 1]
            if constexpr (WRAP) {
                if (a.wrap & 1u) {
                    if ((word >> kStEnd) & 1u) x[2] = RX - 1;
                    if ((word >> (kStEnd + 1)) & 1u) x[0] = 1 - RX;
                }
                if (a.wrap & 2u) {
                    if ((word >> (kStEnd + 2)) & 1u) y[2] = RXY - RX;
                    if ((word >> (kStEnd + 3)) & 1u) y[0] = RX - RXY;
                }
                if (a.wrap & 4u) {
                    if ((word >> (kStEnd + 4)) & 1u) z[2] = R - RXY;
                    if ((word >> (kStEnd + 5)) & 1u) z[0] = RXY - R;
                }
            }
            unroll<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int ex = L::E[i][0];
                if constexpr (i > 0) {
                    int dx = x[ex + 1];
                    // zero-gradient outlet (a link's slot: see tile_links)
                    if constexpr (XB == XBC_OUTFLOW && ex == -1)
                        if (((word >> (kStEnd + 1)) & 1u) && !((word >> i) & 1u)) dx = 0;
                    T v = F[(i - 1) * CAP +
                            (t + m * NT + y[L::E[i][1] + 1] + z[L::E[i][2] + 1] + dx)];
                    if constexpr (XB == XBC_PRESSURE && ex != 0)
                        if (!((word >> i) & 1u) && ((word >> (kStEnd + (ex == 1 ? 0 : 1))) & 1u))
                            v = plus_seam<L, i, kStepTables<T>, ex>(p, v);
                    f[m][i] = v;
                }
            });
        }
        T fi = T(0), fib = T(0);
        LinkCoefT<T> lc{T(0), T(0), T(0), T(0)};
        if ((int)(lk.x & 31u) >= need) {
            lc = lkcoef[lk.y];
            fi = F[lk.z & 0xFFFFu];
            fib = pulled_ibar(lk);
        }
        if (has_more) {
            const uint4 l = a.link[l0 + (uint32_t)(t + NT)];
            if ((int)(l.x & 31u) >= need) {
                later[t] = F[l.z & 0xFFFFu];
                later[t + NT] = pulled_ibar(l);
            }
        }
        __syncthreads();
        // ---- collide
        T* __restrict__ B = out_f[s];
#pragma unroll
        for (int m = 0; m < NPT; ++m) {
            const bool sol = is_solid(st[m]);
            if (st_live(st[m], need)) {
                Macro<L, T> mac;
                collide<L, T, false, kStepTables<T>>(f[m], p, mac);
                unroll<Q>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    if constexpr (i > 0) F[(i - 1) * CAP + t + m * NT] = f[m][i];
                });
            }
            if (B && ((st[m] >> kStMine) & 1u)) {
                // solid nodes as in the single step: NaN where their 64-byte
                // segment of the planes holds a fluid node
                bool store = !sol;
                const uint32_t nn = opaque(n[m]);
                if (sol) {
                    const uint2 wv = nm.wave[nn / 64];
                    store = wave_kind(wv) == WAVE_MIXED && lane_in_live_segment<T>(wv.x, nn & 63u);
                }
                const T nan = (T)__builtin_nan("");
                if (store)
                    unroll<Q>([&](auto I) {
                        constexpr int i = decltype(I)::value;
                        // (a pointer read from LDS: say that it is global)
                        typedef __attribute__((address_space(1))) T G;
                        __builtin_nontemporal_store(sol ? nan : f[m][i], (G*)B + pop_at<Q>(i, nn));
                    });
            }
        }
        // ---- Eq. (213) on the links
        if (n_links) {
            __syncthreads();
            const double ws = wall_scale[s];
            const bool in_window = s >= a.s0 && s < a.s1;
            T* __restrict__ waB = out_wa[s];
            // keeps the conversions to double, and with them the wait for the
            // coefficients, behind the barrier
            asm volatile("" : "+v"(lc.c1), "+v"(lc.c2), "+v"(lc.c3), "+v"(lc.wall));
            auto update = [&](const uint4& l, T gi, T gib, const LinkCoefT<T>& c, double weight,
                              double& sum) {
                const T fpi = F[l.w & 0xFFFFu], fpib = F[l.w >> 16];
                const double v = p.c0 * (double)gi + c.c1 * (double)gib + c.c2 * (double)fpi +
                                 c.c3 * (double)fpib + ws * c.wall;
                T next = (T)v;
                const bool mine = (l.x >> 5) & 1u;
                if (waB && mine) waB[l.y] = next;
                if (p.c1d) {
                    const double c1 = p.c1d[l.y];
                    if (c1 != 0.0) next = (T)((double)next + c1 * (double)pulled_ibar(l));
                }
                F[l.z & 0xFFFFu] = next;
                if (in_window) sum += weight * ((double)fpib + (double)next);
            };
            if ((int)(lk.x & 31u) >= need) update(lk, fi, fib, lc, drag_weight, drag);
            if (has_more) {
                const uint4 l = a.link[l0 + (uint32_t)(t + NT)];
                if ((int)(l.x & 31u) >= need) {
                    const bool in_drag = drags(l);
                    double sum = in_drag ? a.acc[l.y] : 0.0;
                    update(l, later[t], later[t + NT], lkcoef[l.y], in_drag ? weight_of(l) : 0.0, sum);
                    if (in_drag) a.acc[l.y] = sum;
                }
            }
        }
        __syncthreads();
    }
    if (drag_own) a.acc[lk.y] = drag;
}

// ----------------------------------------------------------------------------
// host side

TileLimits tile_limits(const Engine& e) {
    TileLimits lim;
    (void)dispatch(e, [&](auto lat, auto prec, auto) -> hipError_t {
        using S = TileShape<decltype(lat), decltype(prec)>;
        lim.nodes = lim.stride = S::CAP;
        lim.links = S::LINKS;
        lim.per_cu = S::WAVES / 2;
        return hipSuccess;
    });
    return lim;
}

// whether a direction that the lattice moves in wraps inside the region
template <class L>
static bool tile_wraps(const TilePlan& p) {
    return (p.wrap & ((1u << L::D) - 1u)) != 0u;
}

hipError_t tile_setup(const Engine& e) {
    return dispatch(e, [&](auto lat, auto prec, auto xb) -> hipError_t {
        using L = decltype(lat);
        using T = decltype(prec);
        constexpr int XB = decltype(xb)::value;
        const void* kern = tile_wraps<L>(e.tiles) ? (const void*)k_tile_steps<L, T, XB, true>
                                                  : (const void*)k_tile_steps<L, T, XB, false>;
        return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)TileShape<L, T>::LDS);
    });
}

hipError_t launch_tile_steps(Engine& e, const Snapshot& in, const Snapshot* const* out, int steps,
                             const double* ws, const TileDrag& drag) {
    const TilePlan& pl = e.tiles;
    if (steps < 1 || steps > pl.halo) return hipErrorInvalidValue;
    const Grid g = make_grid(e);
    TileArgs a;
    for (int c = 0; c < 3; ++c) {
        a.tile[c] = pl.tile[c];
        a.region[c] = pl.region[c];
    }
    a.blocks = pl.blocks;
    a.per_xcd = (pl.blocks + 7) / 8;
    a.ntile[0] = (uint32_t)pl.ntile[0];
    a.ntile[1] = (uint32_t)pl.ntile[1];
    a.first = e.d_tile_first;
    a.link = e.d_tile_link;
    const uint32_t row = (uint32_t)pl.region[0], plane = row * (uint32_t)pl.region[1];
    a.by_x = ((1u << 22) + row - 1) / row;
    a.by_xy = ((1u << 22) + plane - 1) / plane;
    a.halo = pl.halo;
    a.wrap = pl.wrap;
    a.steps = steps;
    a.acc = drag.acc;
    a.lktag = e.d_lktag;
    a.tag = drag.tag;
    a.s0 = drag.s0;
    a.s1 = drag.s1;
    a.weight = drag.weight;
    for (int s = 0; s < kTileSteps; ++s) a.ws[s] = s < steps ? ws[s] : 1.0;
    return dispatch(e, [&](auto lat, auto prec, auto xb) -> hipError_t {
        using L = decltype(lat);
        using T = decltype(prec);
        TileOut<T> o{};
        for (int s = 0; s < steps; ++s)
            if (out[s]) {
                o.f[s] = (T*)out[s]->f;
                o.wa[s] = (T*)out[s]->wa;
            }
        constexpr int XB = decltype(xb)::value;
        auto kern = tile_wraps<L>(pl) ? k_tile_steps<L, T, XB, true> : k_tile_steps<L, T, XB, false>;
        hipLaunchKernelGGL(kern, dim3(8 * a.per_xcd),
                           dim3(kTileThreads), (TileShape<L, T>::LDS), e.stream, (const T*)in.f,
                           (const T*)in.wa, o, NodeMeta{e.d_info, e.d_wave}, coef_table<T>(e), g,
                           make_params<L, T>(e), a);
        return hipGetLastError();
    });
}

}  // namespace lbe
