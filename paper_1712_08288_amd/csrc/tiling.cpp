// The choice of tiles and the links of their regions (see tiling.hpp).
#include "tiling.hpp"

#include <algorithm>
#include <new>

namespace lbe {

TilePlan tile_plan(const int64_t (&n)[3], const TileLimits& lim, const int (&tile)[3], int halo) {
    TilePlan p;
    int64_t nodes = 1, blocks = 1;
    for (int a = 0; a < 3; ++a) {
        const bool wrap = tile[a] + 2 * halo >= n[a];
        p.tile[a] = wrap ? (int)n[a] : tile[a];
        p.region[a] = wrap ? (int)n[a] : tile[a] + 2 * halo;
        p.ntile[a] = wrap ? 1 : (int)((n[a] + tile[a] - 1) / tile[a]);
        if (wrap) p.wrap |= 1u << a;
        nodes *= p.region[a];
        blocks *= p.ntile[a];
        if (nodes > lim.nodes || p.ntile[a] > 65535 || blocks > (1LL << 24)) return TilePlan{};
    }
    p.blocks = (unsigned)blocks;
    p.halo = halo;
    return p;
}

namespace {

// Microseconds that a launch of plan p takes on 256 CUs, to compare plans by.
// Fitted to D2Q9 launches of 2..12 steps on 64 x 64 to 2048 x 2048 nodes; in
// three dimensions checked against measured launches only (see tile_plans).
constexpr double kCus = 256, kBytesPerUs = 6.2e6, kLaunch = 3.0, kChain = 0.62;

// In two parts, without and with the bytes moved: the first alone rules most
// plans out (a search takes 5 to 40 us, a tenth of what it took with every
// estimate made in full and all plans sorted; lbm_set_geometry 80x42 FP64
// 398 -> 312 us, 301 without tiles).
struct LaunchTime {
    double rounds, at_once, compute;   // compute: microseconds of the steps
};

// What a tile size and a halo make of one direction.
struct Axis {
    int tile, region, ntile;
    bool wrap;
    double line;   // bytes moved for each byte of a row of these tiles
};

LaunchTime launch_steps(const Axis& x, const Axis& y, const Axis& z, int halo, double blocks, int per_cu,
                        double node, int elem) {
    const double X = x.region, Y = y.region, Z = z.region, h = halo;
    // nodes of the waves that compute in some step (waves run along x), the sum
    // of X (Y - 2s or Y) (Z - 2s or Z) over s = 1 .. h
    const double y2 = y.wrap ? 0 : 2, z2 = z.wrap ? 0 : 2;
    const double computed = X * (h * Y * Z - (y2 * Z + z2 * Y) * h * (h + 1) * 0.5 +
                                 y2 * z2 * h * (h + 1) * (2 * h + 1) * (1.0 / 6));
    const double waves = computed / (64 * 4);   // on each SIMD
    const double sharing = std::min<double>(per_cu, std::max(1.0, blocks / kCus));
    const double full = per_cu == 2 ? blocks / (2 * kCus) : blocks / kCus;
    // one block: a chain of LDS and arithmetic latencies; many: the rate at
    // which a SIMD issues the collisions
    const double chain = h * kChain + waves * node * (elem == 8 ? 0.2 : 0.1);
    const double issue = waves * node * sharing * (elem == 8 ? 0.15 : 0.08);
    LaunchTime t;
    t.rounds = std::max(1.0, full);
    t.at_once = std::min<double>(blocks, kCus * per_cu);
    t.compute = std::max(chain, t.rounds * issue);
    return t;
}

}  // namespace

std::vector<TilePlan> tile_plans(const int64_t (&n)[3], const TileLimits& lim, int Q, int D, int elem) {
    constexpr size_t kBest = 8;
    double us[kBest];
    std::vector<TilePlan> best;
    best.reserve(kBest);
    const double nodes = (double)n[0] * (double)n[1] * (double)n[2];
    const double single = std::max(4.0, 2.0 + 2.0 * Q * elem * nodes / kBytesPerUs);
    const double node = Q == 9 ? 1.0 : Q == 15 ? 1.9 : 2.5;
    // A plan has to beat single steps clearly, because the figures compared are
    // estimates (measured: the chosen plan within 6% of the best of those tried
    // on 18 plane domains).  In three dimensions the halo soon costs more than
    // it saves: cubes have plans up to 16^3 (D3Q19 FP64), 18^3 (D3Q15 FP64) and
    // 24^3 (FP32), of 2 or 3 steps, and thin domains.  Measured against the 64
    // steps of a replayed graph, us per step: 16^3 D3Q19 FP64 6.2 and 3.9, FP32
    // 5.8 and 3.1; 24^3 D3Q19 FP32 7.4 and 4.1.  Of the sizes from 8^3 to 48^3
    // and thin ones up to 128x64x2 and 2x88x88, D3Q15 and D3Q19 in both
    // precisions, those with a plan took 0.27 to 0.83 of their single steps.
    double limit = 0.85 * single;
    static const int halos[] = {16, 12, 10, 8, 7, 6, 5, 4, 3, 2};
    static const int sizes[] = {2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 28, 32, 40, 48, 56, 64};
    constexpr int kSizes = sizeof(sizes) / sizeof(sizes[0]);
    for (const int halo : halos) {
        const double per_step = 1.0 / halo;
        if (kLaunch * per_step + kChain >= limit) continue;   // whatever the tile
        // per direction the sizes up to the first that covers the period (larger
        // ones make the same plans)
        Axis axis[3][kSizes];
        int count[3] = {0, 0, 0};
        for (int a = 0; a < 3; ++a)
            for (const int size : sizes) {
                Axis& x = axis[a][count[a]++];
                x.wrap = size + 2 * halo >= n[a];
                x.tile = x.wrap ? (int)n[a] : size;
                x.region = x.wrap ? (int)n[a] : size + 2 * halo;
                x.ntile = x.wrap ? 1 : (int)((n[a] + size - 1) / size);
                // rows are read and written in 64-byte lines that their ends share
                x.line = a == 0 ? 1 + 32.0 / (x.tile * elem) : 1.0;
                if (x.wrap || x.region > lim.nodes || (a == 2 && D == 2)) break;
            }
        for (int i = 0; i < count[0] && axis[0][i].region <= lim.nodes; ++i)
            for (int j = 0; j < count[1]; ++j) {
                const Axis &x = axis[0][i], &y = axis[1][j];
                if ((int64_t)x.region * y.region > lim.nodes) break;
                for (int k = 0; k < count[2]; ++k) {
                    const Axis& z = axis[2][k];
                    const int64_t blocks = (int64_t)x.ntile * y.ntile * z.ntile;
                    if ((int64_t)x.region * y.region * z.region > lim.nodes) break;
                    if (std::max(std::max(x.ntile, y.ntile), z.ntile) > 65535 || blocks > (1LL << 24))
                        continue;
                    const LaunchTime t =
                        launch_steps(x, y, z, halo, (double)blocks, lim.per_cu, node, elem);
                    if ((kLaunch + t.compute) * per_step >= limit) continue;
                    const double region = (double)x.region * y.region * z.region;
                    const double tile = (double)x.tile * y.tile * z.tile;
                    const double move =
                        t.at_once * (region + tile) * Q * elem * x.line * (1.0 / kBytesPerUs);
                    const double total = (kLaunch + t.rounds * move + t.compute) * per_step;
                    if (total >= limit) continue;
                    // into its place among the best, behind equal ones
                    size_t r = best.size() == kBest ? kBest - 1 : best.size();
                    if (r == best.size()) best.emplace_back();
                    for (; r > 0 && total < us[r - 1]; --r) {
                        us[r] = us[r - 1];
                        best[r] = best[r - 1];
                    }
                    us[r] = total;
                    TilePlan& p = best[r];
                    p = TilePlan{};
                    p.halo = halo;
                    const Axis* at[3] = {&x, &y, &z};
                    for (int a = 0; a < 3; ++a) {
                        p.tile[a] = at[a]->tile;
                        p.region[a] = at[a]->region;
                        p.ntile[a] = at[a]->ntile;
                        if (at[a]->wrap) p.wrap |= 1u << a;
                    }
                    p.blocks = (unsigned)blocks;
                    if (best.size() == kBest) limit = us[kBest - 1];
                }
            }
    }
    return best;
}

// (the offsets count links in 32 bits)
constexpr uint32_t kMostLinks = 1u << 31;

static bool place_links(const TilePlan& p, const int64_t (&n)[3], const TileLimits& lim, int Q,
                        const int (*e)[3], const std::vector<int64_t>& node,
                        const std::vector<int8_t>& dir, const std::vector<uint8_t>& ibar_link,
                        bool pressure, bool outflow, TileLinks& out) {
    // per direction and coordinate, the tiles whose region's inside (all but
    // its outermost layer) holds it, with the place in the region, how far that
    // is from the region's edge and whether it is the tile's own: those of
    // coordinate x at [first[x], first[x + 1])
    struct On {
        int tile, loc;
        uint32_t edge, mine;
    };
    std::vector<On> on[3];
    std::vector<uint32_t> first[3];
    for (int a = 0; a < 3; ++a) {
        const int wrap = (int)((p.wrap >> a) & 1u), edge = 1 - wrap;
        auto each = [&](auto&& f) {
            for (int j = 0; j < p.ntile[a]; ++j)
                for (int loc = edge; loc < p.region[a] - edge; ++loc) {
                    const int64_t u = (int64_t)j * p.tile[a] - (wrap ? 0 : p.halo) + loc;
                    const bool mine = wrap || (loc >= p.halo && loc < p.halo + p.tile[a] && u < n[a]);
                    f((size_t)(u < 0 ? u + n[a] : u >= n[a] ? u - n[a] : u),
                      On{j, loc, wrap ? 31u : (uint32_t)std::min(loc, p.region[a] - 1 - loc), mine});
                }
        };
        first[a].assign((size_t)n[a] + 2, 0u);
        each([&](size_t u, On) { ++first[a][u + 2]; });
        for (size_t u = 2; u < first[a].size(); ++u) first[a][u] += first[a][u - 1];
        on[a].resize(first[a].back());
        each([&](size_t u, On o) { on[a][first[a][u + 1]++] = o; });
    }
    std::vector<int> opp((size_t)Q, 0);
    for (int i = 0; i < Q; ++i)
        for (int j = 0; j < Q; ++j)
            if (e[j][0] == -e[i][0] && e[j][1] == -e[i][1] && e[j][2] == -e[i][2]) opp[i] = j;
    // every link's regions in turn, first to count and then to place
    const uint32_t nx = (uint32_t)n[0], ny = (uint32_t)n[1];
    auto each = [&](size_t k, uint32_t (&x)[3], auto&& f) {
        const uint32_t yz = (uint32_t)node[k] / nx;
        x[0] = (uint32_t)node[k] - yz * nx;
        x[2] = yz / ny;
        x[1] = yz - x[2] * ny;
        for (uint32_t c = first[2][x[2]]; c < first[2][x[2] + 1]; ++c)
            for (uint32_t b = first[1][x[1]]; b < first[1][x[1] + 1]; ++b)
                for (uint32_t a = first[0][x[0]]; a < first[0][x[0] + 1]; ++a) {
                    const On at[3] = {on[0][a], on[1][b], on[2][c]};
                    f((size_t)at[0].tile +
                          (size_t)p.ntile[0] * ((size_t)at[1].tile + (size_t)p.ntile[1] * (size_t)at[2].tile),
                      at);
                }
    };
    out.first.assign((size_t)p.blocks + 1, 0u);
    uint32_t x[3];
    for (size_t k = 0; k < node.size(); ++k)
        each(k, x, [&](size_t b, const On*) { ++out.first[b + 1]; });
    out.most = 0;
    for (size_t b = 0; b < p.blocks; ++b) {
        out.most = std::max(out.most, out.first[b + 1]);
        if (out.most > (uint32_t)lim.links || out.first[b] > kMostLinks) return false;
        out.first[b + 1] += out.first[b];
    }
    out.link.reserve((size_t)out.first[p.blocks] + offset_entries(out));
    out.link.resize(out.first[p.blocks]);
    std::vector<uint32_t> next(out.first.begin(), out.first.end() - 1);
    const int stride[3] = {1, p.region[0], p.region[0] * p.region[1]};
    std::vector<int> delta((size_t)Q, 0);   // region index of a node less that of its source
    for (int i = 0; i < Q; ++i)
        for (int a = 0; a < 3; ++a) delta[i] += e[i][a] * stride[a];
    for (size_t k = 0; k < node.size(); ++k) {
        const int i = dir[k], ib = opp[i];
        const bool ibar = ibar_link[k] != 0;
        const int parts = (e[i][0] != 0) + (e[i][1] != 0) + (e[i][2] != 0);
        each(k, x, [&](size_t b, const On* at) {
            const bool at_end = x[0] + 1 == nx;
            const int r = at[0].loc + at[1].loc * stride[1] + at[2].loc * stride[2];
            // region index of x_f - e_j; at the outlet that is a node of the same
            // column unless (x_f, j) is a link, whose own slot is at the periodic
            // neighbour (two links would share the column's)
            auto source = [&](int j, bool link) {
                const bool column = outflow && at_end && e[j][0] == -1 && !link;
                int s = column ? r - delta[j] - 1 : r - delta[j];
                for (int a = column ? 1 : 0; a < 3; ++a)
                    if ((p.wrap >> a) & 1u) {
                        const int loc = at[a].loc - e[j][a];
                        s += loc < 0 ? stride[a] * p.region[a]
                                     : loc >= p.region[a] ? -stride[a] * p.region[a] : 0;
                    }
                return (uint32_t)s;
            };
            auto elem = [&](int j, uint32_t r) { return (uint32_t)(j - 1) * (uint32_t)lim.stride + r; };
            const uint32_t edge = std::min(std::min(at[0].edge, at[1].edge), at[2].edge);
            const uint32_t mine = at[0].mine & at[1].mine & at[2].mine;
            int seam = 0;
            if (pressure && !ibar) {
                if (e[ib][0] == 1 && x[0] == 0) seam = 1;
                if (e[ib][0] == -1 && at_end) seam = -1;
            }
            out.link[next[b]++] = TileLink{
                edge | mine << 5 | (uint32_t)(parts == 1) << 6 | (uint32_t)(e[i][0] + 1) << 7 |
                    (uint32_t)(seam + 1) << 9,
                (uint32_t)k, elem(i, source(i, true)) | elem(ib, source(ib, ibar)) << 16,
                elem(i, (uint32_t)r) | elem(ib, (uint32_t)r) << 16};
        });
    }
    return true;
}

bool tile_links(const TilePlan& p, const int64_t (&n)[3], const TileLimits& lim, int Q,
                const int (*e)[3], const std::vector<int64_t>& node, const std::vector<int8_t>& dir,
                const std::vector<uint8_t>& ibar_link, bool pressure, bool outflow, TileLinks& out) {
    try {
        return place_links(p, n, lim, Q, e, node, dir, ibar_link, pressure, outflow, out);
    } catch (const std::bad_alloc&) {
        out = TileLinks{};
        return false;
    }
}

}  // namespace lbe
