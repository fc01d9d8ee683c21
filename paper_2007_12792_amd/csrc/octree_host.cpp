// Host octree engine: refinement, 26-neighbour periodic 2:1 balance, Morton ordering and the
// ghost-source table (see octfd.h, octree_build).  The tree is an explicit pointer octree; the
// eight children of a node are stored contiguously in Morton child order c = (cz<<2)|(cy<<1)|cx,
// so a depth-first walk visits the leaves in storage order.
//
// Both the balance and the tables rest on one property: the leaves are 2:1 balanced exactly if all 26 neighbour octants of
// every node that has children exist as nodes.  (A leaf with a neighbour two levels coarser has a parent with a neighbour
// octant inside that leaf; the other way round, follow the children on the side of the missing octant down to a leaf.)  So
// only the nodes with children, an eighth of all, are looked at, and the neighbours of a child are children of its
// parent's neighbours, found without a descent from the root.  The rows of the ghost table follow from those neighbours and are
// made where they are needed (table_rows.hpp).  (Tree of 27,756 blocks: 4.8 -> 1.0 ms; with 26 descents
// from the root per leaf for the balance and 27 for its row of the table 23.)
#include "octree_host.hpp"

#include "kernels.hpp"

#include <cstring>
#include <deque>

namespace octfd {
namespace {

constexpr int kQBits = 20;
constexpr int32_t kLeaf = -1, kUnset = -2;

struct Node {
    int32_t first_child;  // >= 0 internal, kLeaf, or kUnset (from_leaves: nothing placed here yet)
    uint32_t level, ix, iy, iz;
    int32_t leaf_id;
    int32_t parent, row;  // row: of a node with children, its place in Octree::inner
};

struct Octree {
    std::vector<Node> nodes;
    std::vector<int32_t> inner;   // the nodes with children, parents first

    Octree() { nodes.push_back(Node{kLeaf, 0, 0, 0, 0, -1, -1, -1}); }

    // turn node n into an internal node with eight children in state `child_state`
    int32_t split(int32_t n, int32_t child_state = kLeaf)
    {
        const Node p = nodes[n];
        const int32_t first = static_cast<int32_t>(nodes.size());
        for (uint32_t c = 0; c < 8; ++c)
            nodes.push_back(Node{child_state, p.level + 1, 2 * p.ix + (c & 1), 2 * p.iy + ((c >> 1) & 1),
                                 2 * p.iz + ((c >> 2) & 1), -1, n, -1});
        nodes[n].row = static_cast<int32_t>(inner.size());
        inner.push_back(n);
        nodes[n].first_child = first;
        return first;
    }

    static uint32_t child_slot(uint32_t l, uint32_t x, uint32_t y, uint32_t z, uint32_t node_level)
    {
        const uint32_t sh = l - node_level - 1;
        return (((z >> sh) & 1) << 2) | (((y >> sh) & 1) << 1) | ((x >> sh) & 1);
    }
};

// periodic distance (2^20-lattice units) from coordinate c to the closed interval [lo, lo+s]
inline int64_t periodic_gap(int64_t c, int64_t lo, int64_t s)
{
    constexpr int64_t kOne = int64_t(1) << kQBits;
    const int64_t t = ((c - lo) % kOne + kOne) % kOne;  // offset of c past lo, going upwards
    if (t <= s) return 0;
    const int64_t up = t - s, down = kOne - t;
    return up < down ? up : down;
}

bool near_seed(const Node& o, const ot_build_params& p)
{
    const int64_t s = int64_t(1) << (kQBits - o.level);
    const int64_t R = p.radius_q20[o.level - p.lmin];
    const int64_t a[3] = {o.ix, o.iy, o.iz};
    for (uint32_t q = 0; q < p.npts; ++q) {
        int64_t d2 = 0;
        for (int d = 0; d < 3; ++d) {
            const int64_t g = periodic_gap(p.pts_q20[3 * q + d], a[d] * s, s);
            d2 += g * g;
        }
        if (d2 < R * R) return true;
    }
    return false;
}

// child_step() as a table
struct ChildSteps {
    ChildStep at[8][kDirs];
    ChildSteps()
    {
        for (int c = 0; c < 8; ++c)
            for (int dir = 0; dir < kDirs; ++dir) at[c][dir] = child_step(c, dir);
    }
};

// Neighbours of every node with children (27, itself in the middle; the root's are the root), in the order of Octree::inner.  A
// missing one lies in a leaf: that leaf is split (and joins the end of the list) or, with may_split = false, the tree is not
// balanced.  A node's parent comes before it, so the parent's neighbours are known and have children by then.
int link_neighbours(Octree& t, bool may_split, std::vector<int32_t>& nbr)
{
    static const ChildSteps steps;
    nbr.assign(kDirs, 0);
    for (size_t r = 1; r < t.inner.size(); ++r) {                    // inner[0] is the root
        const int32_t n = t.inner[r], parent = t.nodes[n].parent;
        const int c = n - t.nodes[parent].first_child;
        const size_t from = static_cast<size_t>(t.nodes[parent].row) * kDirs;
        for (int dir = 0; dir < kDirs; ++dir) {
            const ChildStep s = steps.at[c][dir];
            const int32_t above = nbr[from + s.parent_dir];
            int32_t first = t.nodes[above].first_child;
            if (first < 0) {
                if (!may_split) return OT_E_UNBALANCED;
                first = t.split(above);
            }
            nbr.push_back(first + s.slot);
        }
    }
    return OT_OK;
}

void emit_leaves(Octree& t, int32_t n, std::vector<ot_leaf>& out)
{
    Node& o = t.nodes[n];
    if (o.first_child == kLeaf) {
        o.leaf_id = static_cast<int32_t>(out.size());
        out.push_back(ot_leaf{o.level, o.ix, o.iy, o.iz});
        return;
    }
    const int32_t first = o.first_child;
    for (int c = 0; c < 8; ++c) emit_leaves(t, first + c, out);
}

// What the ghost table is made from, virtual blocks, and which parts of them are read.  The leaves have their ids, `out.nbr` the
// neighbours.
void make_tables(const Octree& t, HostTree& out)
{
    static const ChildSteps steps;
    const size_t nb = out.leaves.size();
    out.node.resize(t.nodes.size());
    for (size_t n = 0; n < t.nodes.size(); ++n) out.node[n] = t.nodes[n].first_child >= 0 ? t.nodes[n].first_child : ~t.nodes[n].leaf_id;
    // A neighbour octant under a leaf is that leaf's child octant: noted in `virt_mask` (per leaf, which of its child octants some
    // block needs) and `coarser`.  Only the children of a node that has a leaf among its neighbours have any.
    struct Coarser { int32_t leaf; int8_t octant, dir; };
    std::vector<Coarser> coarser;
    out.parent.assign(nb, 0);
    out.virt_mask.assign(nb, 0);
    for (size_t r = 0; r < t.inner.size(); ++r) {
        const int32_t first = t.nodes[t.inner[r]].first_child;
        const int32_t* at = &out.nbr[r * kDirs];
        uint32_t leaves = 0;
        for (int dir = 0; dir < kDirs; ++dir) leaves |= static_cast<uint32_t>(out.node[at[dir]] < 0) << dir;
        for (int c = 0; c < 8; ++c) {
            if (out.node[first + c] >= 0) continue;
            out.parent[~out.node[first + c]] = static_cast<int32_t>(8 * r + c);
            if (!leaves) continue;
            for (int dir = 0; dir < kDirs; ++dir) {
                const ChildStep s = steps.at[c][dir];
                if (!((leaves >> s.parent_dir) & 1)) continue;
                const int32_t leaf = ~out.node[at[s.parent_dir]];
                out.virt_mask[leaf] |= static_cast<uint8_t>(1 << s.slot);
                coarser.push_back({leaf, s.slot, static_cast<int8_t>(dir)});
            }
        }
    }
    // virtual blocks, numbered by source leaf, then octant
    out.first_virt.resize(nb);
    out.vblk.clear();
    int32_t n = 0;
    for (size_t s = 0; s < nb; ++s) {
        out.first_virt[s] = n;
        for (int c = 0; c < 8; ++c)
            if ((out.virt_mask[s] >> c) & 1) {
                out.vblk.push_back(static_cast<int32_t>(s));
                out.vblk.push_back(c);
                ++n;
            }
    }
    out.n_virt = n;
    out.vneed.assign(n, 0);
    // a block reads, of its neighbour in direction d, the three layers next to itself along every axis with d != 0
    // and all eight along the others
    auto layers = [](int d) { return d > 0 ? 0x07 : (d < 0 ? 0xE0 : 0xFF); };
    for (const Coarser& e : coarser) {
        const int32_t v = out.first_virt[e.leaf] + __builtin_popcount(static_cast<unsigned>(out.virt_mask[e.leaf]) & ((1u << e.octant) - 1));
        out.vneed[v] |= layers((e.dir / 3) % 3 - 1) | layers(e.dir / 9 - 1) << 8;
    }
}

// the tree's leaves are final but for the balance
int finish(Octree& t, bool may_split, HostTree& out)
{
    if (const int rc = link_neighbours(t, may_split, out.nbr)) return rc;
    out.leaves.clear();
    emit_leaves(t, 0, out.leaves);
    make_tables(t, out);
    make_units(out);
    return OT_OK;
}

}  // namespace

void make_units(HostTree& t)
{
    const size_t nb = t.leaves.size();
    t.units.clear();
    for (size_t b = 0; b < nb;) {
        const ot_leaf& o = t.leaves[b];
        if (b + 1 < nb && !(o.ix & 1)) {
            const ot_leaf& n = t.leaves[b + 1];
            if (n.level == o.level && n.ix == o.ix + 1 && n.iy == o.iy && n.iz == o.iz) {
                t.units.push_back(static_cast<int32_t>(b));
                b += 2;
                continue;
            }
        }
        t.units.push_back(static_cast<int32_t>(b) | kUnitSingle);
        ++b;
    }
}

int build_tree(const ot_build_params& p, HostTree& out)
{
    if (p.lmin < 3 || p.lmax < p.lmin || p.lmax > 19) return OT_E_BADARG;
    if (p.points_per_dim != 8 || p.pad != 3 || p.periodic != 1) return OT_E_UNSUPPORTED;
    if (p.npts && !p.pts_q20) return OT_E_BADARG;
    if (p.lmax > p.lmin && !p.radius_q20) return OT_E_BADARG;
    for (uint32_t q = 0; q < 3 * p.npts; ++q)
        if (p.pts_q20[q] >> kQBits) return OT_E_BADARG;
    // no two points of the periodic cube are further apart than sqrt(3) * 2^19 lattice units; larger radii say
    // nothing more, and beyond 2^31.5 their square would overflow the 64-bit comparison in near_seed()
    for (uint32_t l = p.lmin; l < p.lmax; ++l)
        if (p.radius_q20[l - p.lmin] > (2u << kQBits)) return OT_E_BADARG;

    Octree t;
    std::deque<int32_t> work{0};
    // uniform refinement to lmin, then seed-driven refinement; each node is visited once
    while (!work.empty()) {
        const int32_t n = work.front();
        work.pop_front();
        const Node o = t.nodes[n];
        const bool grow = o.level < p.lmin || (o.level < p.lmax && near_seed(o, p));
        if (!grow) continue;
        const int32_t first = t.split(n);
        for (int c = 0; c < 8; ++c) work.push_back(first + c);
    }
    return finish(t, true, out);
}

int tree_from_leaves(const ot_leaf* leaves, size_t n, HostTree& out)
{
    if (!leaves || n == 0) return OT_E_BADARG;
    Octree t;
    t.nodes[0].first_child = kUnset;
    for (size_t i = 0; i < n; ++i) {
        const ot_leaf& o = leaves[i];
        if (o.level < 3 || o.level > 19 || (o.ix >> o.level) || (o.iy >> o.level) || (o.iz >> o.level))
            return OT_E_BADARG;
        int32_t m = 0;
        while (t.nodes[m].level < o.level) {
            if (t.nodes[m].first_child == kLeaf) return OT_E_INCOMPLETE;      // inside another leaf
            if (t.nodes[m].first_child == kUnset) t.split(m, kUnset);
            m = t.nodes[m].first_child + static_cast<int32_t>(Octree::child_slot(o.level, o.ix, o.iy, o.iz, t.nodes[m].level));
        }
        if (t.nodes[m].first_child != kUnset) return OT_E_INCOMPLETE;        // duplicate or ancestor of a leaf
        t.nodes[m].first_child = kLeaf;
    }
    for (const Node& nd : t.nodes)
        if (nd.first_child == kUnset) return OT_E_INCOMPLETE;                // a gap
    return finish(t, false, out);
}

namespace {
constexpr uint64_t kAround = 0x0000077707770777ull;     // 3^3 of 4^3
// child_step() by where a child's neighbour lies among the 4^3 octants around and in the node; touches() as lists
struct RowTables {
    ChildStep around[64];
    int8_t count[kDirs], slot[kDirs][8];
    RowTables()
    {
        for (int c = 0; c < 8; ++c)
            for (int dir = 0; dir < kDirs; ++dir)
                around[((c >> 2) + dir / 9) * 16 + ((c >> 1 & 1) + dir / 3 % 3) * 4 + (c & 1) + dir % 3] = child_step(c, dir);
        for (int dir = 0; dir < kDirs; ++dir) {
            count[dir] = 0;
            for (int c = 0; c < 8; ++c)
                if (touches(c, dir) && count[dir] < kEntry - 1) slot[dir][count[dir]++] = static_cast<int8_t>(c);
        }
    }
};
}  // namespace

// As table_entry() for every entry.  The neighbours of a node's children, themselves among them, are the 4^3 octants around and in it: looked up once
// for all children, which follow each other in the traversal.  (Trees of 1,296, 27,791 and 102,075 blocks: 0.1, 3.0 and 11.3 ms; a copy of a table
// made with the tree 0.05, 2.4 and 10.7, but then building the trees took 17 and 75 ms longer; table_entry() for each entry 0.65, 13.4 and 47.)
void write_ghost_table(const HostTree& t, int32_t* out)
{
    static const RowTables tables;
    const int32_t* const nodes = t.node.data();
    int32_t entry[64][kEntry], row = -1;             // per axis 0..3: a child's neighbour on that side, or itself
    uint64_t finer = 0;
    for (const int32_t parent : t.parent) {
        if (parent >> 3 != row) {
            row = parent >> 3;
            const int32_t* at = &t.nbr[static_cast<size_t>(row) * kDirs];
            int32_t above[kDirs];
            for (int dir = 0; dir < kDirs; ++dir) above[dir] = nodes[at[dir]];
            finer = 0;
            for (int n = 0; n < 64; ++n) {
                const ChildStep s = tables.around[n];
                const int32_t a = above[s.parent_dir], nd = a < 0 ? a : nodes[a + s.slot];
                int32_t* e = entry[n];
                e[0] = a < 0 ? kCoarser : (nd < 0 ? kSame : kFiner);
                e[1] = ~nd;
                e[2] = e[3] = e[4] = -1;
                finer |= static_cast<uint64_t>(nd >= 0) << n;
            }
        }
        const int first = (parent >> 2 & 1) * 16 + (parent >> 1 & 1) * 4 + (parent & 1);
        for (int n = 0; n < 9; ++n) std::memcpy(out + 3 * kEntry * n, entry[first + n / 3 * 16 + n % 3 * 4], sizeof entry[0] * 3);
        for (uint64_t left = finer >> first & kAround; left; left &= left - 1) {
            const int n = __builtin_ctzll(left), dir = n / 16 * 9 + n / 4 % 4 * 3 + n % 4;
            for (int q = 0; q < tables.count[dir]; ++q) out[dir * kEntry + 1 + q] = ~nodes[~entry[first + n][1] + tables.slot[dir][q]];
        }
        out += kDirs * kEntry;
    }
}

}  // namespace octfd
