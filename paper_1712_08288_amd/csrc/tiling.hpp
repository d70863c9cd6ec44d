// Tiles for launches that take several time steps (tiles.hip): the choice of
// the tile size and the number of steps, in plain C++ (no HIP).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

namespace lbe {

// most steps of one launch on tiles
constexpr int kTileSteps = 16;

// What a block can hold.
struct TileLimits {
    int nodes = 0;          // nodes of a region (tile and halo)
    int links = 0;          // cut links at the nodes inside a region's outermost layer
    int stride = 0;         // LDS elements from one direction's populations to the next
    int per_cu = 0;         // blocks that a CU holds
};

// A region is the tile and `halo` nodes on each side, or, in a direction that
// it would cover anyway, the whole period (bit of `wrap`), without a halo.
struct TilePlan {
    int halo = 0;           // steps of one launch, at most (0: no plan)
    int tile[3] = {0, 0, 0}, region[3] = {0, 0, 0}, ntile[3] = {0, 0, 0};
    uint32_t wrap = 0;
    unsigned blocks = 0;
    unsigned links = 0;     // most cut links of a region, once tile_links has found them
};

// A cut link (x_f, i) as a block meets it: the LDS elements of f_i and f_ibar
// as pulled at x_f and of f'_i and f'_ibar, 16 bits each (population i >= 1 of
// region node r is element (i - 1) stride + r; f_i of a link lies at its solid
// node), its index in the link tables, and bits:
// 0..4 how many nodes x_f is away from the region's edge (31: no edge), 5 a
// node of the tile itself, 6 e_i has one non-zero component, 7..8 e_ix + 1,
// 9..10 sign + 1 of the seam term of the pulled f_ibar.
struct TileLink {
    uint32_t bits, index, pulled, post;
};

// The links of every region, region b's at [first[b], first[b + 1]), at most
// `most` of them.
struct TileLinks {
    std::vector<uint32_t> first;
    std::vector<TileLink> link;
    uint32_t most = 0;
};

// entries of `link` that the offsets would take
inline std::size_t offset_entries(const TileLinks& t) { return (t.first.size() + 3) / 4; }

// The plans that are expected to be faster than single steps, best first.
// Q, D: lattice, elem: bytes of a population value.
std::vector<TilePlan> tile_plans(const int64_t (&n)[3], const TileLimits& lim, int Q, int D, int elem);

// The plan with these tiles; halo = 0 when a region exceeds the nodes a block
// can hold.
TilePlan tile_plan(const int64_t (&n)[3], const TileLimits& lim, const int (&tile)[3], int halo);

// The links of the plan's regions, with room behind them for the offsets
// (offset_entries); false when one has more than a block can hold or there is
// no memory for them.  node, dir: the links in table order, e: the Q velocities, ibar_link:
// whether (x_f, ibar) is a link too; pressure: seam terms in x; outflow: the
// zero-gradient outlet.
bool tile_links(const TilePlan& p, const int64_t (&n)[3], const TileLimits& lim, int Q,
                const int (*e)[3], const std::vector<int64_t>& node, const std::vector<int8_t>& dir,
                const std::vector<uint8_t>& ibar_link, bool pressure, bool outflow, TileLinks& out);

}  // namespace lbe
