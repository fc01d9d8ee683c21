// The ghost table row by row, from the neighbours of nodes with children (see octree_host.cpp).  Shared by the kernel that fills the
// device's table and the host, which hands rows out.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace octfd {

constexpr int kDirs = 27;          // directions (dz+1)*9 + (dy+1)*3 + (dx+1)
constexpr int kEntry = 5;          // {kind, id0..id3}
enum GhostKind : int32_t { kSame = 0, kFiner = 1, kCoarser = 2, kVirtual = 3 };

// What a row is made from: the tree's nodes and, of those with children, the neighbours; about 30 bytes per block, an
// eighteenth of the table.
struct TableSource {
    const int32_t* node;           // [n_nodes] first of eight children, or ~leaf id
    const int32_t* nbr;            // [n_inner][27] nodes: the neighbour octants of the nodes with children
    const int32_t* parent;         // [nb] 8 * (row of the leaf's parent in nbr) + which child it is
    const int32_t* first_virt;     // [nb] the first of the virtual blocks inside a leaf ...
    const uint8_t* virt_mask;      // [nb] ... and which of its child octants have one
};

// For child c = (cz<<2)|(cy<<1)|cx of a node and direction dir: which neighbour of the node holds the child's neighbour octant, and as
// which of its children.
struct ChildStep { int8_t parent_dir, slot; };
__host__ __device__ constexpr ChildStep child_step(int c, int dir)
{
    const int x = (c & 1) + dir % 3 - 1, y = ((c >> 1) & 1) + (dir / 3) % 3 - 1, z = (c >> 2) + dir / 9 - 1;   // -1 .. 2
    const int px = x < 0 ? 0 : (x < 2 ? 1 : 2), py = y < 0 ? 0 : (y < 2 ? 1 : 2), pz = z < 0 ? 0 : (z < 2 ? 1 : 2);
    return {static_cast<int8_t>(pz * 9 + py * 3 + px), static_cast<int8_t>(((z & 1) << 2) | ((y & 1) << 1) | (x & 1))};
}

// Whether child c of the neighbour octant in direction dir touches the block, on the octant's side -dir: along an axis with d = -1 the
// upper children do, with d = +1 the lower ones; axes with d = 0 are free.
__host__ __device__ constexpr bool touches(int c, int dir)
{
    const int d[3] = {dir % 3 - 1, (dir / 3) % 3 - 1, dir / 9 - 1};
    int forced = 0, fixed = 0;
    for (int a = 0; a < 3; ++a)
        if (d[a]) { fixed |= 1 << a; forced |= (d[a] < 0 ? 1 : 0) << a; }
    return (c & fixed) == forced;
}

// entry `dir` of block b; `virt`: a coarser neighbour as the virtual block that stands for it
__host__ __device__ inline void table_entry(const TableSource& t, int64_t b, int dir, bool virt, int32_t (&e)[kEntry])
{
    const int32_t p = t.parent[b];
    const ChildStep s = child_step(p & 7, dir);
    const int32_t above = t.node[t.nbr[static_cast<int64_t>(p >> 3) * kDirs + s.parent_dir]];
    e[1] = e[2] = e[3] = e[4] = -1;
    if (above < 0) {
        const int32_t leaf = ~above;
        e[0] = virt ? kVirtual : kCoarser;
        e[1] = leaf;
        if (virt) e[1] = t.first_virt[leaf] + __builtin_popcount(t.virt_mask[leaf] & ((1u << s.slot) - 1));
        return;
    }
    const int32_t nd = t.node[above + s.slot];
    if (nd < 0) {
        e[0] = kSame;
        e[1] = ~nd;
        return;
    }
    // the children that touch the block, x first, then y, then z (ascending Morton order)
    e[0] = kFiner;
    int n = 1;
    for (int c = 0; c < 8; ++c)
        if (touches(c, dir) && n < kEntry) e[n++] = ~t.node[nd + c];
}

}  // namespace octfd
