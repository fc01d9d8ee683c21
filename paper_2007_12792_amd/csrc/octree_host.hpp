// Host-side octree engine of liboctfd: pointer octree, 2:1 balance, Morton-order
// traversal and the ghost-source table.  No device code here.
#pragma once
#include <cstdint>
#include <vector>

#include "octfd.h"
#include "table_rows.hpp"

namespace octfd {

struct HostTree {
    std::vector<ot_leaf> leaves;   // Morton order
    // What the rows of the ghost table are made from (TableSource)
    std::vector<int32_t> node, nbr, parent, first_virt;
    std::vector<uint8_t> virt_mask;
    TableSource source() const { return {node.data(), nbr.data(), parent.data(), first_virt.data(), virt_mask.data()}; }
    // "Virtual blocks".  Where the same-level neighbour octant of a block does not exist because its parent L is
    // a leaf, the ghost values in that direction are interpolated inside L, and what they are depends only on L's
    // data and on the fine position inside L, not on which block asks.  Such an octant can therefore be filled
    // once, like a child of L ("virtual block"), after which the blocks around it read it
    // exactly like a neighbour of their own level.
    //   vblk    [n_virt][2]        per virtual block {source leaf id, child octant (ox | oy<<1 | oz<<2)}, ordered by
    //                              source leaf (Morton order), then octant
    //   n_virt                     number of virtual blocks
    //   vneed   [n_virt]           which y rows (bits 0..7) and z planes (bits 8..15) of a virtual block any block reads: the
    //                              union, per axis, over the blocks that have it as a neighbour.  The fill writes only
    //                              those (whole x rows of them); the rest of a virtual block is never read.
    std::vector<int32_t> vblk, vneed;
    int64_t n_virt = 0;
    // Work units of the two-block kernel of the 24-field system, in Morton order: the first block of every two
    // leaves that are the lower and upper x child of one parent (they follow each other in storage), and, flagged
    // with kUnitSingle, every other block (a leaf whose x sibling is subdivided).  Every block belongs to exactly one unit.
    std::vector<int32_t> units;
};

// Each returns an OT_* status.  The ghost table itself is not kept: the device makes its own from source(), write_ghost_table() hands it out.
int build_tree(const ot_build_params& p, HostTree& out);
int tree_from_leaves(const ot_leaf* leaves, size_t n, HostTree& out);
// the ghost table, to out[nb][27][5]
void write_ghost_table(const HostTree& t, int32_t* out);
void make_units(HostTree& t);

}  // namespace octfd
