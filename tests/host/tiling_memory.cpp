// Host-only driver for the tiles' link tables (csrc/tiling.cpp) when memory runs
// out, built by tests/test_host_tiling_memory.py: every allocation in turn is
// refused.  tile_links must then report that there is no table, as it does for
// regions with too many links, and never let the exception out (its caller is a
// C entry point); with memory it leaves room for the offsets behind the links.
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "../../paper_1712_08288_amd/csrc/tiling.hpp"

static long left_over = -1;   // allocations until one is refused (negative: none is)

void* operator new(size_t n) {
    if (left_over == 0) throw std::bad_alloc();
    if (left_over > 0) --left_over;
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main() {
    const int E2[9][3] = {{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {-1, 0, 0}, {0, -1, 0},
                          {1, 1, 0}, {-1, 1, 0}, {-1, -1, 0}, {1, -1, 0}};
    const int64_t n[3] = {200, 120, 1};
    lbe::TileLimits lim;
    lim.nodes = lim.stride = 1024;
    lim.links = 1024;
    lim.per_cu = 2;
    std::vector<int64_t> node;
    std::vector<int8_t> dir;
    std::vector<uint8_t> ibar;
    for (int64_t k = 0; k < n[0] * n[1]; k += 17)   // (any links will do)
        for (int i = 1; i < 9; ++i) {
            node.push_back(k);
            dir.push_back((int8_t)i);
            ibar.push_back((uint8_t)(i & 1));
        }
    const lbe::TilePlan p = lbe::tile_plans(n, lim, 9, 2, 8).at(0);
    int refused = 0;
    for (long k = 0; k < 1000; ++k) {
        lbe::TileLinks t;
        left_over = k;
        const bool ok = lbe::tile_links(p, n, lim, 9, E2, node, dir, ibar, false, false, t);
        left_over = -1;
        if (!ok) {
            if (!t.first.empty() || !t.link.empty()) return 1;
            ++refused;
            continue;
        }
        if (t.first.size() != p.blocks + 1u || t.link.size() != t.first.back() || t.link.empty() ||
            t.link.capacity() < t.link.size() + lbe::offset_entries(t))
            return 2;
        std::printf("ok: %d refusals\n", refused);
        return refused >= 8 ? 0 : 3;
    }
    return 4;
}
