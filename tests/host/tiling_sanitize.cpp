// Host-only driver for the tiles of multi-step launches (csrc/tiling.cpp),
// built with the address and undefined-behaviour sanitizers by
// tests/test_host_tiling.py.  On seeded random domains and plans it moves
// labelled populations as a block does -- every population of the region in
// its own LDS element, cut links at their solid nodes -- and checks that each
// node is stored by exactly one block, that every element a step reads lies in
// the array and holds the population the whole domain's pull would read there.
#include <algorithm>
#include <cstdio>
#include <map>
#include <random>
#include <string>
#include <tuple>
#include <vector>

#include "../../paper_1712_08288_amd/csrc/tiling.hpp"

namespace {

const int E2[9][3] = {{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {-1, 0, 0}, {0, -1, 0},
                      {1, 1, 0}, {-1, 1, 0}, {-1, -1, 0}, {1, -1, 0}};
const int E3[15][3] = {{0, 0, 0},  {1, 0, 0},  {-1, 0, 0}, {0, 1, 0},  {0, -1, 0},
                       {0, 0, 1},  {0, 0, -1}, {1, 1, 1},  {-1, 1, 1}, {1, -1, 1},
                       {-1, -1, 1}, {1, 1, -1}, {-1, 1, -1}, {1, -1, -1}, {-1, -1, -1}};

int failures = 0, plans = 0, links_seen = 0;

void check(bool ok, const std::string& what) {
    if (!ok && ++failures < 20) std::printf("FAIL: %s\n", what.c_str());
}

int64_t wrap(int64_t u, int64_t n) { return ((u % n) + n) % n; }

void run(std::mt19937_64& rng, int Q, const int (*e)[3], const int64_t (&n)[3], bool outflow,
         bool pressure, const lbe::TilePlan& p, const lbe::TileLimits& lim) {
    const int64_t N = n[0] * n[1] * n[2];
    std::vector<char> solid((size_t)N, 0);
    for (auto& s : solid) s = rng() % 5 == 0;
    if (outflow)
        for (int64_t k = 0; k < N; k += n[0]) solid[(size_t)k] = 1;
    auto source = [&](int64_t k, int i) {   // node that the pull of i at k reads
        int64_t x = k % n[0] - e[i][0];
        if (outflow) x = std::min(std::max<int64_t>(x, 0), n[0] - 1);
        return wrap(x, n[0]) + n[0] * (wrap((k / n[0]) % n[1] - e[i][1], n[1]) +
                                       n[1] * wrap(k / (n[0] * n[1]) - e[i][2], n[2]));
    };
    std::vector<int> opp((size_t)Q);
    for (int i = 0; i < Q; ++i)
        for (int j = 0; j < Q; ++j)
            if (e[i][0] == -e[j][0] && e[i][1] == -e[j][1] && e[i][2] == -e[j][2]) opp[i] = j;
    std::vector<int64_t> node;
    std::vector<int8_t> dir;
    std::vector<uint8_t> ibar;
    std::map<std::pair<int64_t, int>, uint32_t> index;
    for (int64_t k = 0; k < N; ++k)
        for (int i = 1; i < Q; ++i)
            if (!solid[(size_t)k] && solid[(size_t)source(k, i)]) {
                index[{k, i}] = (uint32_t)node.size();
                node.push_back(k);
                dir.push_back((int8_t)i);
                ibar.push_back(solid[(size_t)source(k, opp[i])]);
            }
    lbe::TileLinks tl;
    const bool ok = lbe::tile_links(p, n, lim, Q, e, node, dir, ibar, pressure, outflow, tl);
    if (!ok) return;
    ++plans;
    check(tl.first.size() == (size_t)p.blocks + 1 && tl.first.back() == tl.link.size(), "offsets");
    std::vector<int> stored((size_t)N, 0);
    const int R = p.region[0] * p.region[1] * p.region[2];
    for (unsigned b = 0; b < p.blocks; ++b) {
        const int at[3] = {(int)(b % p.ntile[0]), (int)(b / p.ntile[0] % p.ntile[1]),
                           (int)(b / p.ntile[0] / p.ntile[1])};
        std::vector<int64_t> glob((size_t)R);
        std::vector<int> edge((size_t)R), mine((size_t)R);
        // labels: (node k, direction i) as k Q + i, links -1 - index
        std::vector<int64_t> lds((size_t)(Q - 1) * lim.stride, INT64_MIN);
        for (int r = 0; r < R; ++r) {
            const int loc[3] = {r % p.region[0], r / p.region[0] % p.region[1],
                                r / (p.region[0] * p.region[1])};
            int64_t g[3];
            edge[r] = 31;
            mine[r] = 1;
            for (int a = 0; a < 3; ++a) {
                const bool w = (p.wrap >> a) & 1u;
                const int64_t u = (int64_t)at[a] * p.tile[a] - (w ? 0 : p.halo) + loc[a];
                check(u >= -n[a] && u < 2 * n[a], "one period suffices");
                g[a] = wrap(u, n[a]);
                if (w) continue;
                edge[r] = std::min(edge[r], std::min(loc[a], p.region[a] - 1 - loc[a]));
                mine[r] = mine[r] && loc[a] >= p.halo && loc[a] < p.halo + p.tile[a] && u < n[a];
            }
            glob[r] = g[0] + n[0] * (g[1] + n[1] * g[2]);
            if (mine[r]) ++stored[(size_t)glob[r]];
            check(!mine[r] || edge[r] >= p.halo, "a tile's node is `halo` nodes inside");
            if (!solid[(size_t)glob[r]])
                for (int i = 1; i < Q; ++i) lds[(size_t)(i - 1) * lim.stride + r] = glob[r] * Q + i;
        }
        std::map<std::tuple<int, int>, const lbe::TileLink*> of;   // by region node, direction
        for (uint32_t l = tl.first[b]; l < tl.first[b + 1]; ++l) {
            const lbe::TileLink& t = tl.link[l];
            ++links_seen;
            const int i = dir[t.index], r = (int)(t.post & 0xFFFFu) - (i - 1) * lim.stride;
            check(r >= 0 && r < R && glob[r] == node[t.index], "link's node");
            if (r < 0 || r >= R) return;
            check((int)(t.bits & 31u) == edge[r] && (int)((t.bits >> 5) & 1u) == mine[r] && edge[r] >= 1,
                  "edge and tile bits");
            check((int)((t.bits >> 7) & 3u) - 1 == e[i][0], "x component");
            check(((t.bits >> 6) & 1u) == (unsigned)(e[i][0] * e[i][0] + e[i][1] * e[i][1] +
                                                      e[i][2] * e[i][2] == 1), "axis bit");
            const int64_t x = node[t.index] % n[0];
            const int ib = opp[i];
            const int seam = !pressure || ibar[t.index] ? 0
                             : e[ib][0] == 1 && x == 0 ? 1 : e[ib][0] == -1 && x + 1 == n[0] ? -1 : 0;
            check((int)((t.bits >> 9) & 3u) - 1 == seam, "seam sign");
            const size_t slot = t.pulled & 0xFFFFu;
            check(slot < lds.size() && lds[slot] == INT64_MIN, "a link's slot is its own");
            if (slot < lds.size()) lds[slot] = -1 - (int64_t)t.index;
            check(of.emplace(std::make_tuple(r, i), &t).second, "a link once per region");
            check((t.post >> 16) == (uint32_t)((ib - 1) * lim.stride + r), "f'_ibar");
        }
        // the first step's pull at every node inside the region
        for (int r = 0; r < R; ++r) {
            if (solid[(size_t)glob[r]] || edge[r] < 1) continue;
            const int loc[3] = {r % p.region[0], r / p.region[0] % p.region[1],
                                r / (p.region[0] * p.region[1])};
            const bool end = glob[r] % n[0] + 1 == n[0];
            for (int i = 1; i < Q; ++i) {
                const auto it = index.find({glob[r], i});
                const bool link = it != index.end();
                int q = 0;
                for (int a = 2; a >= 0; --a) {
                    int u = loc[a] - e[i][a];
                    if (a == 0 && outflow && end && e[i][0] == -1 && !link) u = loc[0];
                    if ((p.wrap >> a) & 1u) u = (int)wrap(u, p.region[a]);
                    check(u >= 0 && u < p.region[a], "pull inside the region");
                    q = q * p.region[a] + u;
                }
                const int64_t got = lds[(size_t)(i - 1) * lim.stride + q];
                check(got == (link ? -1 - (int64_t)it->second : source(glob[r], i) * Q + i), "pull");
                const auto lt = of.find(std::make_tuple(r, opp[i]));   // this is that link's f_ibar
                if (lt != of.end())
                    check((lt->second->pulled >> 16) == (uint32_t)((i - 1) * lim.stride + q), "f_ibar");
            }
        }
    }
    for (int64_t k = 0; k < N; ++k) check(stored[(size_t)k] == 1, "every node in one tile");
}

}  // namespace

int main() {
    std::mt19937_64 rng(7);
    for (int trial = 0; trial < 210; ++trial) {
        const bool three = trial % 3 == 0;
        int64_t n[3] = {1 + (int64_t)(rng() % 40), 1 + (int64_t)(rng() % 30), 1};
        if (three)
            for (auto& v : n) v = 1 + (int64_t)(rng() % 14);
        const int bc = (int)(rng() % 3);
        if (bc == 1 && n[0] < 2) n[0] = 2;
        lbe::TileLimits lim;
        lim.nodes = lim.stride = three ? 512 : 1024;
        lim.links = trial % 7 == 0 ? 60 : 4096;
        lim.per_cu = 2;
        const int tile[3] = {1 + (int)(rng() % 16), 1 + (int)(rng() % 16), 1 + (int)(rng() % 6)};
        const lbe::TilePlan p = lbe::tile_plan(n, lim, tile, 1 + (int)(rng() % (three ? 4 : 8)));
        if (p.halo)
            run(rng, three ? 15 : 9, three ? E3 : E2, n, bc == 1, bc == 2, p, lim);
        // the chosen plans keep to the limits
        for (const lbe::TilePlan& c : lbe::tile_plans(n, lim, three ? 15 : 9, three ? 3 : 2, 8)) {
            check(c.halo >= 2 && c.halo <= lbe::kTileSteps &&
                      c.region[0] * c.region[1] * c.region[2] <= lim.nodes, "limits");
            if (trial % 10 == 0) run(rng, three ? 15 : 9, three ? E3 : E2, n, bc == 1, bc == 2, c, lim);
        }
    }
    check(plans > 100 && links_seen > 10000, "coverage");
    if (failures) return 1;
    std::printf("ok: %d plans, %d links\n", plans, links_seen);
    return 0;
}
