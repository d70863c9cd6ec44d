// Adjoint (reverse-mode) step of the forward kernel.
//
// The forward map of one step t -> t+1 at fluid node y is
//   g(y)   = C(f(y, t))                         collision, Eq. (22a)
//   f_i(y + e_i, t+1) = g_i(y)                  advection, Eq. (22b)
//   f_i(y, t+1) = c0 f_i(y,t) + c1 f_ibar(y,t) + c2 g_i(y) + c3 g_ibar(y)
//                 + c4 * 3 w_i rho0 e_i.phi     cut link (y, i), Eq. (213)
// With lambda(t+1) = dJ/df(., t+1) the reverse step computes, per node,
//   mu_i(y)  = dJ/dg_i(y): lambda_i(y + e_i, t+1) when that node pulls from y,
//              plus c2 / c3 times the node's own link adjoints,
//   lambda(y, t) = (dC/df)^T mu + c0 / c1 times the own link adjoints,
// where (dC/df)^T mu = mu - (I - J^T) M^T R M mu, R = diag(s_k / |M_k|^2),
// and J_ij = d f^eq_i / d f_j = w_i [1 + (3 e_i + 9 (e_i.u) e_i - 3 u).e_j]
// (derivative of Eq. (42)), so that (J^T v)_j = a + b.e_j with
// a = sum_i w_i v_i and b = sum_i w_i v_i (3 e_i + 9 (e_i.u) e_i - 3 u).
// Gradients accumulated on the way, in double (the per-link ones by the
// lanes that carry the links, the others in per-block sums):
//   dJ/dgamma_k += a_k (dc1 f_ibar + dc2 g_i + dc3 g_ibar + ws dwall),
//   dJ/dphi_k   += a_k ws c4 3 w_i rho0 e_i,
//   dJ/dg       += sum_i mu_i 3 w_i rho0 e_i,
//   dJ/ds_k     += -(M mu)_k (M (f - f^eq))_k / |M_k|^2,
// where a_k is the adjoint of the link value f_i(y, t+1) and ws the
// wall-data factor of step t.  The wall terms share the factor a_k ws, so
// per link only two sums are kept, gq_k = sum a_k (dc1 f_ibar + dc2 g_i +
// dc3 g_ibar) and gs_k = sum a_k ws; the gradients are formed from them
// when read (k_link_finish).
#pragma once

#include "engine.hpp"
#include "kernels.hpp"
#include "params.hpp"

namespace lbe {

// Node indices of x + e (the node that pulls from this one along e).
template <int XB>
struct Push {
    uint32_t xt[3];
    uint32_t row[3][3];
    bool x_out;   // outflow: no node at x = nx (e_x = +1 from the last column)

    __device__ __forceinline__ Push(const Grid& g, const NodePos& p) {
        const uint32_t xm = p.ix == 0 ? g.nx - 1 : p.ix - 1;
        const uint32_t xp = p.ix + 1 == g.nx ? 0u : p.ix + 1;
        xt[0] = xm;       // e_x = -1 lands at x - 1
        xt[1] = p.ix;
        xt[2] = xp;       // e_x = +1 lands at x + 1
        x_out = (XB == XBC_OUTFLOW) && (p.ix + 1 == g.nx);
        const uint32_t ys[3] = {p.iy == 0 ? g.ny - 1 : p.iy - 1, p.iy,
                                p.iy + 1 == g.ny ? 0u : p.iy + 1};
        const uint32_t zs[3] = {p.iz == 0 ? g.nz - 1 : p.iz - 1, p.iz,
                                p.iz + 1 == g.nz ? 0u : p.iz + 1};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int c = 0; c < 3; ++c) row[a][c] = g.nx * (ys[a] + g.ny * zs[c]);
    }

    template <class L, int I>
    __device__ __forceinline__ uint32_t dst() const {
        return xt[L::E[I][0] + 1] + row[L::E[I][1] + 1][L::E[I][2] + 1];
    }
    // outflow: the last column also pulls its -x populations from here
    template <class L, int I>
    __device__ __forceinline__ uint32_t dst_clamped(uint32_t ix) const {
        return ix + row[L::E[I][1] + 1][L::E[I][2] + 1];
    }
};

struct AdjArgs {
    int obj_kind;        // LBM_OBJ_* of the header
    int obj_tag;
    double w_force;      // weight of this step's drag term (0 outside window)
    double w_ux;         // weight of d(mean u_x)/df_j = e_jx * w_ux
    int want_ds;
    // pressure drop: dJ/df_j(x) = a_in [x = x_in] - a_out [x = x_out] for
    // every j at fluid nodes (a_* include the step's weight and c_s^2)
    uint32_t x_in, x_out;
    double a_in, a_out;
};

// The per-link gradient sums of the sweep (see the header): gq at g[k] and
// gs at g[L1 + k], with the gamma-derivatives of the coefficients they
// need.  In the kernel that reads step records g is instead the step's run
// of a_k (one per link), summed later by k_link_sums.  Pointers are few on
// purpose: every kernel argument the adjoint keeps costs scalar registers,
// which bound its occupancy.
struct LinkGrad {
    const LinkDeriv* deriv;
    double* g;
    uint32_t L1;     // max(L, 1): the stride of the runs of g and of a record
};

// One step's contribution of link k with adjoint a_k (drag term included)
// and the forward values f_ibar(y, t), f'_i(y, t), f'_ibar(y, t).
template <class T>
__device__ __forceinline__ void link_gradient(const LinkGrad& lg, uint32_t k, double ak, T fib,
                                              T fpi, T fpib, double ws) {
    const double d1 = lg.deriv[k].d1, d2 = lg.deriv[k].d2, d3 = lg.deriv[k].d3;
    lg.g[k] += ak * (d1 * (double)fib + d2 * (double)fpi + d3 * (double)fpib);
    lg.g[lg.L1 + k] += ak * ws;
}

// Lattice data of a direction known only at run time (link lanes): e_d, w_d
// and the opposite direction.
template <class L>
__device__ __forceinline__ void dir_data(int d, int (&e)[3], double& w, int& opp) {
    unroll<L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if (i == d) {
            e[0] = L::E[i][0];
            e[1] = L::E[i][1];
            e[2] = L::E[i][2];
            w = L::W[i];
            opp = TAB<L>.opp[i];
        }
    });
}

// Walk a node's cut links in direction order (links are sorted by node,
// then direction, so the k-th set bit of the mask is link nl.base + k).  For
// the wave's first 64 links the two LDS values of the link, st.v[A][k] and
// st.v[B][k], are read one direction ahead of their use, with the index
// clamped to the slab instead of a divergent branch around the access, so
// that the reads overlap; own(I, va, vb, k) consumes them, direct(I, k)
// handles a link past the 64th.
template <class L, class T, int A, int B, class Own, class Direct>
__device__ __forceinline__ void walk_links(const NodeLinks& nl, LinkStage<T>& st, Own&& own,
                                           Direct&& direct) {
    uint32_t k = nl.base;
    uint32_t kk = k < 64u ? k : 63u;
    T a_next = st.v[A][kk], b_next = st.v[B][kk];
    unroll<L::Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (i > 0) {
            const uint32_t bit = (nl.mask >> i) & 1u;
            const T va = a_next, vb = b_next;
            const uint32_t k1 = k + bit;
            if constexpr (i + 1 < L::Q) {
                kk = k1 < 64u ? k1 : 63u;
                a_next = st.v[A][kk];
                b_next = st.v[B][kk];
            }
            if (bit) {
                if (k < 64u) own(I, va, vb, k);
                else direct(I, k);
            }
            k = k1;
        }
    });
}

// Sums over the lanes of a wave of N values each.  At every level the two
// halves of the lanes exchange one half of the values each, so 17 exchanges
// reduce the 15 rates of D3Q19 where a reduction of one value after the other
// takes 90; afterwards a lane holds one sum.
template <int N, int M>
__device__ __forceinline__ void wave_sums(double* v, uint32_t lane) {
    if constexpr (N == 1) {
        v[0] += __shfl_xor(v[0], M, 64);
        if constexpr (M > 1) wave_sums<1, M / 2>(v, lane);
    } else {
        constexpr int H = (N + 1) / 2;
        const bool hi = (lane & M) != 0u;
#pragma unroll
        for (int c = 0; c < H; ++c) {
            const double a = v[c], b = c + H < N ? v[c + H] : 0.0;
            v[c] = (hi ? b : a) + __shfl_xor(hi ? a : b, M, 64);
        }
        static_assert(M > 1, "at most 64 values");
        wave_sums<H, M / 2>(v, lane);
    }
}
// the value whose sum wave_sums leaves in a lane, or -1 (none, or another
// lane's as well)
template <int N>
__device__ __forceinline__ int wave_sum_column(uint32_t lane) {
    int n = N, at = 0, valid = N;
    bool first = true;
#pragma unroll
    for (uint32_t m = 32; m > 0; m >>= 1) {
        const bool hi = (lane & m) != 0u;
        if (n == 1) {
            first = first && !hi;
            continue;
        }
        const int h = (n + 1) / 2;
        at += hi ? h : 0;
        valid = hi ? valid - h : min(valid, h);
        n = h;
    }
    return first && valid > 0 ? at : -1;
}

// Links past the 64th of a mixed wave are handled by the lane of their node y
// (the first 64 go through the wave's LDS slab).  The adjoint a_k of link
// k = (y, i), drag term dfx included.
template <class L, class T, int i>
__device__ __forceinline__ double own_link_adjoint(uint32_t k, const T* __restrict__ lam_in,
                                                   uint32_t n, const int32_t* __restrict__ lktag,
                                                   const AdjArgs& a, double& dfx) {
    double ak = (double)ldp<L::Q>(lam_in, i, n);
    dfx = 0.0;
    if (a.obj_kind == 1 && L::E[i][0] != 0 && lktag[k] == a.obj_tag) {
        // drag: (e_ibar)_x (f'_ibar(y,t) + f_i(y,t+1))
        dfx = -(double)L::E[i][0] * a.w_force;
        ak += dfx;
    }
    return ak;
}

// The terms of such a link that bypass the collision: c0 a_k onto
// lambda_i(y, t) and c1 a_k onto lambda_ibar(y, t), added to mu after its
// moments are taken (a_k read again: these links are rare).
template <class L, class T, int i>
__device__ __forceinline__ void own_link_bypass(uint32_t k, const T* __restrict__ lam_in,
                                                uint32_t n,
                                                const LinkCoefT<T>* __restrict__ lkcoef,
                                                const int32_t* __restrict__ lktag,
                                                const Params<L, T>& p, const AdjArgs& a,
                                                T (&mu)[L::Q]) {
    constexpr int ib = TAB<L>.opp[i];
    double dfx;
    const double ak = own_link_adjoint<L, T, i>(k, lam_in, n, lktag, a, dfx);
    mu[i] += (T)(p.c0 * ak);
    mu[ib] += (T)(lkcoef[k].c1 * ak);
}

// The waves of the adjoint launch, slot s < count (s = 4 blockIdx.x + wave in
// the block), each as {id, kind | links << 2, first link, 0} (node
// n = 64 id + lane) so that one scalar load brings all of it.  wpr = nx / 64
// when 64 divides nx (each wave lies in one row), else 0.
struct WaveList {
    const uint4* ent;
    uint32_t count;
    uint32_t wpr;
};

template <bool ROWS>
__device__ __forceinline__ NodePos node_of_wave(const Grid& g, const WaveList& wl, uint32_t w,
                                                uint32_t lane, bool active) {
    NodePos p;
    p.n = w * 64u + lane;
    p.in = active && p.n < g.N;
    if constexpr (ROWS) {
        const uint32_t row = w / wl.wpr;
        p.ix = (w - row * wl.wpr) * 64u + lane;
        p.iz = row / g.ny;
        p.iy = row - p.iz * g.ny;
    } else {
        const uint32_t row = p.n / g.nx;
        p.ix = p.n - row * g.nx;
        p.iz = row / g.ny;
        p.iy = row - p.iz * g.ny;
    }
    return p;
}

// One launch covers the non-idle waves in memory order.  Plain and mixed
// waves take separate paths from the start.  Mixed waves handle their cut
// links cooperatively (see LinkStage): the link lanes read the link data
// and a_k = lambda_i(y, t+1) (plus the drag term) with coalesced loads and
// hand c2 a_k, c3 a_k (+ drag), c0 a_k and c1 a_k to the node's lane
// through LDS; the node's lane hands back f_ibar(y, t), from which with
// a_k and the forward step's stored f'_i(y, t), f'_ibar(y, t) the link
// lanes add the link's gradient sums.
// UM: the forward state enters the collision adjoint only through its
// velocity (the equilibrium's Jacobian depends on u alone and is applied to
// moments, which the transform back needs anyway), so with the rate
// gradients off the kernel reads u(y, t) recorded by the forward step (D
// planes of U) instead of pulling the Q populations of f(y, t), and the
// link values of the gradients come from the same step record: A, wa and
// nxt are not read.
// Bound by HBM traffic and the mixed waves' latencies on large domains, by the
// length of a launch on small ones.  The transforms by row factors, the
// Jacobian on moments, the rate sums without divisions and wave_sums by halves
// took a reverse step (node and link kernels, us) from 615 to 518 at 256^3 FP32
// on records, 287 to 262 at 256x256x64 FP64, 750 to 604 at 256x256x128 FP32 with
// the rate gradients and 85 to 72 at 96x64x64 FP64 with them and the replay.
// Waves per SIMD asked of the compiler, where it stops just short of them:
// FP64 on step records 4 (130 VGPRs fitted into 128 made the reverse step 3.5%
// faster at 256^3); with the rate gradients FP64 D3 3, FP32 D3 4 and FP32 D2 6.
// The others are left to the compiler (forcing more waves on them spilled more
// and was slower).
template <class L, class T>
constexpr int adjoint_waves(bool want_ds, bool um) {
    if (sizeof(T) == 8) return um ? 4 : L::D == 3 ? 3 : 1;
    return want_ds ? (L::D == 3 ? 4 : 6) : 1;
}
template <class L, class T, int XB, bool WANT_DS, bool ROWS, bool UM>
__global__ void __launch_bounds__(BX)
__attribute__((amdgpu_waves_per_eu(adjoint_waves<L, T>(WANT_DS, UM))))
k_adjoint(const T* __restrict__ A, StepRecord<T> rec, const T* __restrict__ wa,
          const T* __restrict__ nxt,
          const T* __restrict__ lam_in, T* __restrict__ lam_out,
          NodeMeta nm, WaveList wl, const LinkCoefT<T>* __restrict__ lkcoef,
          const int32_t* __restrict__ lktag,
          const uint8_t* __restrict__ lkdir, const int32_t* __restrict__ lknode,
          LinkGrad lgr, double* __restrict__ gglob, Grid g, Params<L, T> p, AdjArgs a) {
    constexpr int Q = L::Q, D = L::D, NP = NPAIR<L>;
    static_assert(!(UM && WANT_DS), "the rate gradients need the forward populations");
    constexpr int NC = D + Q;                 // layout of the per-block sums
    constexpr int NK = Q - D - 1;             // rows with a rate
    __shared__ LinkStage<T> stage[BX / 64];
    // the link lanes' a_k, parked while the node's work runs (registers are
    // scarcest there), and the f_ibar(y, t) that the nodes' lanes hand them
    __shared__ double ak_park[BX / 64][64];
    __shared__ T fib_park[BX / 64][UM ? 1 : 64];
    const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t slot = blockIdx.x * (BX / 64) + wid;
    const bool active = slot < wl.count;
    const uint4 wm = active ? wl.ent[slot] : uint4{0u, 0u, 0u, 0u};
    const uint32_t w = __builtin_amdgcn_readfirstlane(wm.x);
    const uint32_t wx = __builtin_amdgcn_readfirstlane(wm.y);
    const uint32_t nlw = wave_links(uint2{wx, 0u});
    const uint32_t wbase = __builtin_amdgcn_readfirstlane(wm.z);
    const NodePos pos = node_of_wave<ROWS>(g, wl, w, lane, active);
    LinkStage<T>& st = stage[wid];
    double acc[D];
#pragma unroll
    for (int c = 0; c < D; ++c) acc[c] = 0.0;
    double ds_sum = 0.0;                      // of the rate row of wave_sum_column
    // What a read-modify-write at the kernel's end needs is read in advance
    // where that costs no occupancy (reverse step reading states, D2Q9 FP64
    // 512x256: 16.1 -> 15.3 us); on records it costs a wave per SIMD (66
    // registers instead of 63) and gains nothing, D3 FP64 spills for it.
    constexpr bool EARLY = !UM && (sizeof(T) == 4 || D == 2);
    double* const sums = gglob + (size_t)blockIdx.x * NC;
    double before = 0.0;
    // (thread c adds gradient column c below D, then the rows with a rate)
    int column = (int)threadIdx.x < D ? (int)threadIdx.x : -1;
    double scale = 3.0 * p.rho0_d;
    if constexpr (WANT_DS) {
        int c = D;
        unroll<Q>([&](auto K) {
            constexpr int kk = decltype(K)::value;
            if constexpr (!L::conserved(kk))
                if ((int)threadIdx.x == c++) {
                    column = D + kk;
                    scale = -1.0 / (double)TAB<L>.norm[kk];
                }
        });
    }
    if (EARLY && column >= 0) before = sums[column];

    // One wave's work.  Plain and mixed waves take separate paths from the
    // start (their own loads included), so that each path's registers are
    // allocated as in a kernel of its own.  Plain waves are 64 fluid nodes
    // inside the grid.
    auto run = [&](auto mixed_c) {
        constexpr bool MX = decltype(mixed_c)::value;
        // mixed waves: the link lanes' indices come first (small coalesced
        // loads), so that the gathers that depend on them can be issued before
        // the node loads below return
        const bool link_lane = MX && lane < nlw && lane < 64u;
        const uint32_t kl = wbase + lane;
        int ld_dir = 0;
        uint32_t ld_node = 0;
        if (link_lane) {
            ld_dir = lkdir[kl];
            ld_node = (uint32_t)lknode[kl];
        }

        // loads that do not depend on the node's metadata: the planes of the
        // forward pull and the adjoint gathers lambda_i(y + e_i, t+1) (entries
        // of solid or absent neighbours are read and then discarded)
        T f[Q], lg[Q], uv[3] = {T(0), T(0), T(0)};
        const Push<XB> ps(g, pos);
        // plain waves are 64 fluid nodes inside the grid; in mixed waves the
        // lanes of 64-byte plane segments without fluid nodes neither read nor
        // write
        const bool live = !MX || (pos.in && lane_in_live_segment<T>(wx, lane));
        if (live) {
            if constexpr (UM) {
                for (int a = 0; a < D; ++a) uv[a] = ld(rec.u + (size_t)a * g.S, pos.n);
            } else {
                pull_planes<L, T, XB>(A, g, pos, p, NodeLinks{0u, 0u}, f);
            }
            unroll<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                lg[i] = ldp<Q>(lam_in, i, i == 0 ? pos.n : ps.template dst<L, i>());
            });
        } else {
            unroll<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                f[i] = T(0);
                lg[i] = T(0);
            });
        }

        // one node per lane; PLAIN: the whole wave is fluid without cut links.  In
        // a mixed wave nl.base is relative to the wave's first link and f already
        // holds the link slots; its solid lanes go along (sol), so that the wave
        // stays whole for the sums and writes whole lines of lam_out: they add
        // nothing and store NaN (nothing reads lambda at solid nodes; partial
        // lines cost HBM read-modify-write cycles).
        auto node = [&](auto plain_c, const NodeLinks& nl, bool sol) {
            constexpr bool PLAIN = decltype(plain_c)::value;
            // forward state f(y, t) and its velocity (UM: the recorded one)
            T sp[NP], dp[NP];
            T rho = 0, j[3] = {0, 0, 0}, u[3];
            if constexpr (UM) {
                u[0] = uv[0];
                u[1] = uv[1];
                u[2] = uv[2];
            } else {
                pair_split<L, T>(f, sp, dp);
                conserved_of<L, T>(f[0], sp, dp, rho, j);
                u[0] = j[0] * p.inv_rho0;
                u[1] = j[1] * p.inv_rho0;
                u[2] = j[2] * p.inv_rho0;
            }
            // own cut links, read from states: f_ibar(y, t) goes to the link
            // lane, which takes the gradients (past the 64th taken here)
            if constexpr (!PLAIN && !UM) {
                if (nl.mask) {
                    uint32_t k = nl.base;
                    unroll<Q>([&](auto I) {
                        constexpr int i = decltype(I)::value;
                        constexpr int ib = TAB<L>.opp[i];
                        if constexpr (i > 0) {
                            const uint32_t bit = (nl.mask >> i) & 1u;
                            if (bit) {
                                if (k < 64u) {
                                    fib_park[wid][k] = f[ib];
                                } else {
                                    double dfx;
                                    const double ak = own_link_adjoint<L, T, i>(
                                        wbase + k, lam_in, pos.n, lktag, a, dfx);
                                    link_gradient(lgr, wbase + k, ak, f[ib],
                                                  ldp<Q>(nxt, i, pos.n), ldp<Q>(nxt, ib, pos.n),
                                                  p.wall_scale);
                                }
                            }
                            k += bit;
                        }
                    });
                }
            }
            // M (f - f^eq), so that f and its pairs die here
            T neq[Q];
            if constexpr (WANT_DS) nonequilibrium_of<L, T>(f[0], sp, dp, j, p.inv_rho0, neq);

            // mu_i(y) = dJ/df'_i(y): lambda_i(y + e_i, t+1) where that node pulls
            T mu[Q];
            unroll<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int ib = TAB<L>.opp[i];
                if constexpr (i == 0) {
                    mu[i] = lg[0];
                } else {
                    bool lost = (nl.mask >> ib) & 1u;     // y + e_i is solid
                    if constexpr (XB == XBC_OUTFLOW && L::E[i][0] == 1) lost = lost || ps.x_out;
                    mu[i] = lost ? T(0) : lg[i];
                    if constexpr (XB == XBC_OUTFLOW && L::E[i][0] == -1) {
                        if (ps.x_out && !sol) {
                            const uint32_t n2 = ps.template dst_clamped<L, i>(pos.ix);
                            if (!is_solid(nm.info[n2])) mu[i] += ldp<Q>(lam_in, i, n2);
                        }
                    }
                }
            });

            // own cut links: Eq. (213) reversed and the drag terms
            if constexpr (!PLAIN) {
                if (nl.mask) {
                    walk_links<L, T, 0, 1>(
                        nl, st,
                        [&](auto I, T va, T vb, uint32_t) {
                            constexpr int i = decltype(I)::value;
                            constexpr int ib = TAB<L>.opp[i];
                            mu[i] += va;
                            mu[ib] += vb;
                        },
                        [&](auto I, uint32_t k) {
                            constexpr int i = decltype(I)::value;
                            constexpr int ib = TAB<L>.opp[i];
                            double dfx;
                            const double ak = own_link_adjoint<L, T, i>(wbase + k, lam_in, pos.n,
                                                                        lktag, a, dfx);
                            const LinkCoefT<T> c = lkcoef[wbase + k];
                            mu[ib] += (T)dfx;
                            mu[i] += (T)(c.c2 * ak);
                            mu[ib] += (T)(c.c3 * ak);
                            // the step's a_k run; k_link_sums adds the terms
                            if constexpr (UM) lgr.g[wbase + k] = ak;
                        });
                }
            }

            // collision adjoint: lambda = mu - v + J^T v + (c0, c1 link terms),
            // v = M^T R M mu
            T smu[NP], dmu[NP];
            pair_split<L, T>(mu, smu, dmu);
            T qm[Q];
            moments_of<L, T>(mu[0], smu, dmu, qm);
            if constexpr (WANT_DS) {
                // dJ/ds_k -= (M mu)_k (M (f - f^eq))_k / |M_k|^2 (the factor
                // on the sums: a division here would cost more than the rest),
                // summed over the wave at once, so that one value is held
                double prod[NK];
                int c = 0;
                unroll<Q>([&](auto K) {
                    constexpr int kk = decltype(K)::value;
                    if constexpr (!L::conserved(kk))
                        prod[c++] = !PLAIN && sol ? 0.0 : (double)qm[kk] * (double)neq[kk];
                });
                wave_sums<NK, 32>(prod, lane);
                ds_sum = prod[0];
            }

            // dJ/dg += 3 rho0 sum_i w_i e_i mu_i (pair form: w_i e_i (mu_i - mu_ibar)),
            // summed over the node in T, accumulated over nodes in double
            // (taken here in mixed waves, so that dmu dies before the link
            // terms below; at the end in plain waves)
            auto add_dg = [&]() {
                T sg3[3] = {0, 0, 0};
                unroll<NP>([&](auto P) {
                    constexpr int pp = decltype(P)::value;
                    constexpr int i = DER<L>.pi[pp];
                    const T t = T(L::W[i]) * dmu[pp];
                    macc<L::E[i][0]>(sg3[0], t);
                    macc<L::E[i][1]>(sg3[1], t);
                    macc<L::E[i][2]>(sg3[2], t);
                });
#pragma unroll
                for (int al = 0; al < D; ++al)
                    acc[al] += !PLAIN && sol ? 0.0 : (double)sg3[al];
            };
            if constexpr (!PLAIN) add_dg();

            // the link terms that bypass the collision (c0 a_k onto
            // lambda_i(y, t), c1 a_k onto lambda_ibar(y, t)) join mu now that
            // its moments are taken, so that they need no registers of their own
            if constexpr (!PLAIN) {
                if (nl.mask) {
                    walk_links<L, T, 2, 3>(
                        nl, st,
                        [&](auto I, T va, T vb, uint32_t) {
                            constexpr int i = decltype(I)::value;
                            constexpr int ib = TAB<L>.opp[i];
                            mu[i] += va;
                            mu[ib] += vb;
                        },
                        [&](auto I, uint32_t k) {
                            constexpr int i = decltype(I)::value;
                            own_link_bypass<L, T, i>(wbase + k, lam_in, pos.n, lkcoef, lktag, p,
                                                     a, mu);
                        });
                }
            }
            T r[Q];
            unroll<Q>([&](auto K) {
                constexpr int kk = decltype(K)::value;
                r[kk] = L::conserved(kk) ? T(0) : qm[kk] * p.rate[kk];
            });
            // J^T v = (d m^eq / df)^T r = as + b.e_j: with m^eq_k = A_k drho + B_k.j
            // + C_k (jj) / rho0 (Derived), as = sum_k A_k r_k and
            // b = sum_k r_k (B_k + d (C_k (jj) / rho0) / dj), taken from the
            // moments instead of the populations of v (a third of the operations)
            T as, b[3];
            {
                Sum<T> sa, sb[3], sc[6];
                unroll<Q>([&](auto K) {
                    constexpr int kk = decltype(K)::value;
                    if constexpr (!L::conserved(kk)) {
                        if constexpr (DER<L>.A[kk] != 0.0) sa.term(T(DER<L>.A[kk]), r[kk]);
                        unroll<3>([&](auto X) {
                            constexpr int x = decltype(X)::value;
                            if constexpr (DER<L>.B[kk][x] != 0.0)
                                sb[x].term(T(DER<L>.B[kk][x]), r[kk]);
                        });
                        unroll<6>([&](auto C) {
                            constexpr int c = decltype(C)::value;
                            if constexpr (DER<L>.C[kk][c] != 0.0)
                                sc[c].term(T(DER<L>.C[kk][c]), r[kk]);
                        });
                    }
                });
                as = sa.v;
                b[0] = sb[0].v + (T(2) * sc[0].v * u[0] + sc[3].v * u[1] + sc[5].v * u[2]);
                b[1] = sb[1].v + (sc[3].v * u[0] + T(2) * sc[1].v * u[1] + sc[4].v * u[2]);
                b[2] = sb[2].v + (sc[5].v * u[0] + sc[4].v * u[1] + T(2) * sc[2].v * u[2]);
            }
            T e0, ev[NP], od[NP];
            back_transform<L, T>(r, e0, ev, od);
            const T wux = (T)a.w_ux;
            // pressure drop: the same term for every population of the node
            if (a.obj_kind == 3)
                as += (T)((pos.ix == a.x_in ? a.a_in : 0.0) - (pos.ix == a.x_out ? a.a_out : 0.0));
            auto finish = [&](auto J, T v) {
                constexpr int jd = decltype(J)::value;
                T out = mu[jd] - v + as;
                macc<L::E[jd][0]>(out, b[0]);
                macc<L::E[jd][1]>(out, b[1]);
                macc<L::E[jd][2]>(out, b[2]);
                if (a.obj_kind == 2) macc<L::E[jd][0]>(out, wux);
                if constexpr (!PLAIN)
                    if (sol) out = (T)__builtin_nan("");
                if (PLAIN || live) stp_nt<Q>(lam_out, jd, pos.n, out);
            };
            finish(std::integral_constant<int, 0>{}, e0);
            unroll<NP>([&](auto P) {
                constexpr int pp = decltype(P)::value;
                constexpr int i = DER<L>.pi[pp];
                constexpr int ib = TAB<L>.opp[i];
                finish(std::integral_constant<int, i>{}, ev[pp] + od[pp]);
                finish(std::integral_constant<int, ib>{}, ev[pp] - od[pp]);
            });
            if constexpr (PLAIN) add_dg();
        };

        if constexpr (!MX) {
            node(std::true_type{}, NodeLinks{0u, 0u}, false);
        } else {
            // link lanes: the link's adjoint a_k = lambda_i(y, t+1) and (reading
            // states) the forward step's stored f'_i(y, t), f'_ibar(y, t)
            int le[3] = {0, 0, 0}, lib = 0;
            double lw = 0.0;
            double ak = 0.0;
            T fpi = T(0), fpib = T(0);
            // reading states: the sums and derivatives the gradients need at the end
            double gq = 0.0, gs = 0.0, d1 = 0.0, d2 = 0.0, d3 = 0.0;
            auto read_sums = [&]() {
                gq = lgr.g[kl];
                gs = lgr.g[lgr.L1 + kl];
                d1 = lgr.deriv[kl].d1;
                d2 = lgr.deriv[kl].d2;
                d3 = lgr.deriv[kl].d3;
            };
            LinkCoefT<T> c{T(0), T(0), T(0), T(0)};
            if (link_lane) {
                dir_data<L>(ld_dir, le, lw, lib);
                c = lkcoef[kl];
                ak = (double)ldp<Q>(lam_in, ld_dir, ld_node);
                if constexpr (!UM) {
                    fpi = ldp<Q>(nxt, ld_dir, ld_node);
                    fpib = ldp<Q>(nxt, lib, ld_node);
                    if constexpr (EARLY) read_sums();
                }
            }
            const uint32_t info = live ? nm.info[pos.n] : kInfoSolid;
            const bool sol = is_solid(info);
            const NodeLinks nl = sol ? NodeLinks{0u, 0u} : node_links(info, 0u);
            if constexpr (!UM) {
                // forward state: the link slots of the recorded step
                const T wa0 = lane < nlw ? wa[wbase + lane] : T(0);
                wave_link_values<L, T>(wa, wbase, lane, wa0, nl, st, f);
                if (p.c1d) complete_two_node<L, T>(p.c1d + wbase, nl, f);
            }
            // link lanes: the pieces of mu and lambda(y, t) that a_k feeds
            if (link_lane) {
                double dfx = 0.0;
                if (a.obj_kind == 1 && le[0] != 0 && lktag[kl] == a.obj_tag) {
                    // drag: (e_ibar)_x (f'_ibar(y,t) + f_i(y,t+1))
                    dfx = -(double)le[0] * a.w_force;
                    ak += dfx;
                }
                st.v[0][lane] = (T)(c.c2 * ak);
                st.v[1][lane] = (T)(c.c3 * ak + dfx);
                st.v[2][lane] = (T)(p.c0 * ak);
                st.v[3][lane] = (T)(c.c1 * ak);
                // the link's gradient sums: with records a_k is stored into the
                // step's run and k_link_sums adds the terms; else they are added
                // once the node's lane has handed back f_ibar(y, t)
                if constexpr (UM)
                    lgr.g[kl] = ak;
                else
                    ak_park[wid][lane] = ak;
            }
            wave_lds_sync();
            node(std::false_type{}, nl, sol);
            wave_lds_sync();
            if constexpr (!UM)
                if (link_lane) {
                    if constexpr (!EARLY) read_sums();
                    const double ak_l = ak_park[wid][lane];
                    lgr.g[kl] = gq + ak_l * (d1 * (double)fib_park[wid][lane] + d2 * (double)fpi +
                                             d3 * (double)fpib);
                    lgr.g[lgr.L1 + kl] = gs + ak_l * p.wall_scale;
                }
        }
    };
    if (active) {
        if ((__builtin_amdgcn_readfirstlane(wm.y) & 3u) == WAVE_PLAIN)
            run(std::false_type{});
        else
            run(std::true_type{});
    }

    // the waves' sums, then the block's
    __shared__ double part[BX / 64][D + NK];
    wave_sums<D, 32>(acc, lane);
    const int col = wave_sum_column<D>(lane), row = wave_sum_column<NK>(lane);
    if (col >= 0) part[wid][col] = acc[0];
    if constexpr (WANT_DS)
        if (row >= 0) part[wid][D + row] = ds_sum;
    __syncthreads();
    if (column >= 0) {
        double s = 0.0;
        for (int w = 0; w < BX / 64; ++w) s += part[w][threadIdx.x];
        if (!EARLY) before = sums[column];
        sums[column] = before + s * scale;
    }
}

// The node kernel of one reverse step for the handle's precision, x boundary
// and sweep, one lattice per translation unit.
struct AdjointLaunch {
    const Snapshot *fwd, *next;     // null when rec is given
    const void* rec;
    const void* lam_in;
    void* lam_out;
    LinkGrad links;
    AdjArgs args;
};

template <class L>
hipError_t launch_adjoint_nodes(const Engine& e, const AdjointLaunch& a) {
    const uint32_t wpr = e.nx % 64 == 0 ? (uint32_t)(e.nx / 64) : 0u;
    const WaveList waves{e.d_wact, (uint32_t)e.n_wact, wpr};
    if (!waves.count) return hipSuccess;
    auto go = [&](auto prec, auto xb) -> hipError_t {
        using T = decltype(prec);
        constexpr int XB = decltype(xb)::value;
        const bool um = a.rec != nullptr;
        auto kern = a.args.want_ds ? (wpr ? k_adjoint<L, T, XB, true, true, false>
                                          : k_adjoint<L, T, XB, true, false, false>)
                    : um           ? (wpr ? k_adjoint<L, T, XB, false, true, true>
                                          : k_adjoint<L, T, XB, false, false, true>)
                                   : (wpr ? k_adjoint<L, T, XB, false, true, false>
                                          : k_adjoint<L, T, XB, false, false, false>);
        hipLaunchKernelGGL(kern, dim3((waves.count + BX / 64 - 1) / (BX / 64)), dim3(BX), 0, e.stream,
                           um ? nullptr : (const T*)a.fwd->f,
                           um ? record_at<T>(e, a.rec) : StepRecord<T>{},
                           um ? nullptr : (const T*)a.fwd->wa, um ? nullptr : (const T*)a.next->f,
                           (const T*)a.lam_in, (T*)a.lam_out, NodeMeta{e.d_info, e.d_wave}, waves,
                           coef_table<T>(e), e.d_lktag, e.d_lkdir, e.d_lknode, a.links, e.d_gglob,
                           make_grid(e), make_params<L, T>(e), a.args);
        return hipGetLastError();
    };
    auto by_xbc = [&](auto prec) -> hipError_t {
        switch (e.xbc) {
            case XBC_PRESSURE: return go(prec, std::integral_constant<int, XBC_PRESSURE>{});
            case XBC_OUTFLOW: return go(prec, std::integral_constant<int, XBC_OUTFLOW>{});
            default: return go(prec, std::integral_constant<int, XBC_PERIODIC>{});
        }
    };
    return e.precision == 0 ? by_xbc(double{}) : by_xbc(float{});
}
extern template hipError_t launch_adjoint_nodes<D2Q9>(const Engine&, const AdjointLaunch&);
extern template hipError_t launch_adjoint_nodes<D3Q15>(const Engine&, const AdjointLaunch&);
extern template hipError_t launch_adjoint_nodes<D3Q19>(const Engine&, const AdjointLaunch&);

}  // namespace lbe
