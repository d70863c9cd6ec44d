// The choice of tiles and the links of their regions (see tiling.hpp).
#include "tiling.hpp"

#include <algorithm>

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
// Fitted to D2Q9 launches of 2..12 steps on 64 x 64 to 2048 x 2048 nodes.
constexpr double kCus = 256, kBytesPerUs = 6.2e6;

double launch_us(const TilePlan& p, const TileLimits& lim, int Q, int elem) {
    double region = 1, tile = 1, computed = 0;
    for (int a = 0; a < 3; ++a) {
        region *= p.region[a];
        tile *= p.tile[a];
    }
    // nodes of the waves that compute in some step: waves run along x
    for (int s = 1; s <= p.halo; ++s) {
        double c = p.region[0];
        for (int a = 1; a < 3; ++a) c *= p.region[a] - ((p.wrap >> a) & 1u ? 0 : 2 * s);
        computed += c;
    }
    const double waves = computed / (64 * 4);   // on each SIMD
    const double node = Q == 9 ? 1.0 : Q == 15 ? 1.9 : 2.5;
    const double sharing = std::min<double>(lim.per_cu, std::max(1.0, p.blocks / kCus));
    const double rounds = std::max(1.0, p.blocks / (kCus * lim.per_cu));
    // rows are read and written in 64-byte lines that their ends share
    const double line = 1 + 32.0 / (p.tile[0] * elem);
    const double at_once = std::min<double>(p.blocks, kCus * lim.per_cu);
    const double move = at_once * (region + tile) * Q * elem * line / kBytesPerUs;
    // one block: a chain of LDS and arithmetic latencies; many: the rate at
    // which a SIMD issues the collisions
    const double chain = p.halo * 0.62 + waves * node * (elem == 8 ? 0.2 : 0.1);
    const double issue = waves * node * sharing * (elem == 8 ? 0.15 : 0.08);
    return 3.0 + rounds * move + std::max(chain, rounds * issue);
}

}  // namespace

std::vector<TilePlan> tile_plans(const int64_t (&n)[3], const TileLimits& lim, int Q, int D, int elem) {
    struct Rated {
        double us;
        TilePlan p;
    };
    std::vector<Rated> all;
    const double nodes = (double)n[0] * (double)n[1] * (double)n[2];
    const double single = std::max(4.0, 2.0 + 2.0 * Q * elem * nodes / kBytesPerUs);
    // Regions over 512 nodes in three dimensions lose more to the halo than a
    // launch costs, so on domains that are not thin no plan passes the test
    // against single steps below; it asks for a clear gain, because the figures
    // compared are estimates (measured: the chosen plan within 6% of the best
    // of those tried on 18 domains).
    static const int halos[] = {2, 3, 4, 5, 6, 7, 8, 10, 12, 16};
    static const int sizes[] = {2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 28, 32, 40, 48, 56, 64};
    for (const int halo : halos)
        for (const int x : sizes) {
            if (x + 2 * halo > lim.nodes) break;
            for (const int y : sizes) {
                if (std::min<int64_t>(n[0], x + 2 * halo) * std::min<int64_t>(n[1], y + 2 * halo) >
                    lim.nodes)
                    break;
                for (const int z : sizes) {
                    if (D == 2 && z != sizes[0]) break;
                    const int tile[3] = {x, y, z};
                    const TilePlan p = tile_plan(n, lim, tile, halo);
                    if (!p.halo) break;
                    const double us = launch_us(p, lim, Q, elem) / halo;
                    if (us < 0.85 * single) all.push_back(Rated{us, p});
                    if (p.wrap & 4u) break;   // larger tiles give the same plan
                }
                if (y + 2 * halo >= n[1]) break;
            }
            if (x + 2 * halo >= n[0]) break;
        }
    std::stable_sort(all.begin(), all.end(), [](const Rated& a, const Rated& b) { return a.us < b.us; });
    std::vector<TilePlan> out;
    for (const Rated& r : all) {
        if (out.size() == 8) break;
        out.push_back(r.p);
    }
    return out;
}

bool tile_links(const TilePlan& p, const int64_t (&n)[3], const TileLimits& lim, int Q,
                const int (*e)[3], const std::vector<int64_t>& node, const std::vector<int8_t>& dir,
                const std::vector<uint8_t>& ibar_link, bool pressure, bool outflow, TileLinks& out) {
    // per direction and coordinate, the tiles whose region's inside (all but
    // its outermost layer) holds it, with the place in the region
    struct On {
        int tile, loc;
    };
    std::vector<std::vector<On>> on[3];
    for (int a = 0; a < 3; ++a) {
        on[a].resize((size_t)n[a]);
        const bool wrap = (p.wrap >> a) & 1u;
        for (int j = 0; j < p.ntile[a]; ++j)
            for (int loc = wrap ? 0 : 1; loc < p.region[a] - (wrap ? 0 : 1); ++loc) {
                const int64_t u = (int64_t)j * p.tile[a] - (wrap ? 0 : p.halo) + loc;
                on[a][(size_t)(((u % n[a]) + n[a]) % n[a])].push_back(On{j, loc});
            }
    }
    std::vector<int> opp((size_t)Q, 0);
    for (int i = 0; i < Q; ++i)
        for (int j = 0; j < Q; ++j)
            if (e[j][0] == -e[i][0] && e[j][1] == -e[i][1] && e[j][2] == -e[i][2]) opp[i] = j;
    // every link's regions in turn, first to count and then to place
    auto each = [&](auto&& f) {
        for (size_t k = 0; k < node.size(); ++k) {
            const int64_t x[3] = {node[k] % n[0], (node[k] / n[0]) % n[1], node[k] / (n[0] * n[1])};
            for (const On& z : on[2][(size_t)x[2]])
                for (const On& y : on[1][(size_t)x[1]])
                    for (const On& xx : on[0][(size_t)x[0]]) {
                        const On at[3] = {xx, y, z};
                        f(k, x,
                          (size_t)xx.tile + (size_t)p.ntile[0] *
                                                ((size_t)y.tile + (size_t)p.ntile[1] * (size_t)z.tile),
                          at);
                    }
        }
    };
    out.first.assign((size_t)p.blocks + 1, 0u);
    each([&](size_t, const int64_t*, size_t b, const On*) { ++out.first[b + 1]; });
    for (size_t b = 0; b < p.blocks; ++b) {
        if (out.first[b + 1] > (uint32_t)lim.links) return false;
        out.first[b + 1] += out.first[b];
    }
    out.link.resize(out.first[p.blocks]);
    std::vector<uint32_t> next(out.first.begin(), out.first.end() - 1);
    each([&](size_t k, const int64_t* x, size_t b, const On* at) {
        const int i = dir[k], ib = opp[i];
        const bool at_end = x[0] + 1 == n[0];
        // region index of x_f - e_j; at the outlet that is a node of the same
        // column unless (x_f, j) is a link, whose own slot is at the periodic
        // neighbour (two links would share the column's)
        auto source = [&](int j, bool link) {
            int r = 0;
            for (int a = 2; a >= 0; --a) {
                int loc = at[a].loc - e[j][a];
                if (a == 0 && outflow && at_end && e[j][0] == -1 && !link) loc = at[0].loc;
                if ((p.wrap >> a) & 1u) loc = (loc + p.region[a]) % p.region[a];
                r = r * p.region[a] + loc;
            }
            return (uint32_t)r;
        };
        auto elem = [&](int j, uint32_t r) { return (uint32_t)(j - 1) * (uint32_t)lim.stride + r; };
        uint32_t r = 0, edge = 31;
        bool mine = true;
        int parts = 0;
        for (int a = 2; a >= 0; --a) {
            r = r * (uint32_t)p.region[a] + (uint32_t)at[a].loc;
            parts += e[i][a] != 0;
            if ((p.wrap >> a) & 1u) continue;
            edge = std::min(edge, (uint32_t)std::min(at[a].loc, p.region[a] - 1 - at[a].loc));
            mine = mine && at[a].loc >= p.halo && at[a].loc < p.halo + p.tile[a] &&
                   (int64_t)at[a].tile * p.tile[a] + at[a].loc - p.halo < n[a];
        }
        int seam = 0;
        if (pressure && !ibar_link[k]) {
            if (e[ib][0] == 1 && x[0] == 0) seam = 1;
            if (e[ib][0] == -1 && at_end) seam = -1;
        }
        out.link[next[b]++] = TileLink{
            edge | (uint32_t)mine << 5 | (uint32_t)(parts == 1) << 6 | (uint32_t)(e[i][0] + 1) << 7 |
                (uint32_t)(seam + 1) << 9,
            (uint32_t)k, elem(i, source(i, true)) | elem(ib, source(ib, ibar_link[k] != 0)) << 16,
            elem(i, r) | elem(ib, r) << 16};
    });
    return true;
}

}  // namespace lbe
