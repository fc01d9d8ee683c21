// Host octree engine: refinement, 26-neighbour periodic 2:1 balance, Morton ordering and the
// ghost-source table (see octfd.h, octree_build).  The tree is an explicit pointer octree; the
// eight children of a node are stored contiguously in Morton child order c = (cz<<2)|(cy<<1)|cx,
// so a depth-first walk visits the leaves in storage order.
//
// Both the balance and the tables rest on one property: the leaves are 2:1 balanced exactly if all 26 neighbour octants of
// every node that has children exist as nodes.  (A leaf with a neighbour two levels coarser has a parent with a neighbour
// octant inside that leaf; the other way round, follow the children on the side of the missing octant down to a leaf.)  So
// only the nodes with children, an eighth of all, are looked at, and the neighbours of a child are children of its
// parent's neighbours, found without a descent from the root.  (Tree of 27,756 blocks with its tables, these in huge
// pages: 23 -> 4.8 ms; 26 descents from the root per leaf for the balance and 27 for its table row took most of it.)
#include "octree_host.hpp"

#include "kernels.hpp"

#include <deque>

namespace octfd {
namespace {

constexpr int kQBits = 20;
constexpr int32_t kLeaf = -1, kUnset = -2;

struct Node {
    int32_t first_child;  // >= 0 internal, kLeaf, or kUnset (from_leaves: nothing placed here yet)
    uint32_t level, ix, iy, iz;
    int32_t leaf_id;
};

struct Octree {
    std::vector<Node> nodes;

    Octree() { nodes.push_back(Node{kLeaf, 0, 0, 0, 0, -1}); }

    // turn node n into an internal node with eight children in state `child_state`
    int32_t split(int32_t n, int32_t child_state = kLeaf)
    {
        const Node p = nodes[n];
        const int32_t first = static_cast<int32_t>(nodes.size());
        for (uint32_t c = 0; c < 8; ++c)
            nodes.push_back(Node{child_state, p.level + 1, 2 * p.ix + (c & 1), 2 * p.iy + ((c >> 1) & 1),
                                 2 * p.iz + ((c >> 2) & 1), -1});
        nodes[n].first_child = first;
        return first;
    }

    static uint32_t child_slot(uint32_t l, uint32_t x, uint32_t y, uint32_t z, uint32_t node_level)
    {
        const uint32_t sh = l - node_level - 1;
        return (((z >> sh) & 1) << 2) | (((y >> sh) & 1) << 1) | ((x >> sh) & 1);
    }

    // deepest existing node on the path from the root towards octant (l; x, y, z), depth <= l
    int32_t descend(uint32_t l, uint32_t x, uint32_t y, uint32_t z) const
    {
        int32_t n = 0;
        while (nodes[n].first_child >= 0 && nodes[n].level < l)
            n = nodes[n].first_child + static_cast<int32_t>(child_slot(l, x, y, z, nodes[n].level));
        return n;
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

// Splits leaves until every node with children has its 26 neighbour octants, finest level first: what a node at level l
// asks for is split at coarser levels only.  inner[l]: the nodes of level l that have children.
void balance(Octree& t, std::vector<int32_t> (&inner)[21])
{
    for (int l = 20; l >= 1; --l) {
        const uint32_t mask = (1u << l) - 1;
        for (size_t q = 0; q < inner[l].size(); ++q) {
            const Node o = t.nodes[inner[l][q]];
            for (int dir = 0; dir < kDirs; ++dir) {
                const uint32_t x = (o.ix + (dir % 3 - 1)) & mask, y = (o.iy + ((dir / 3) % 3 - 1)) & mask, z = (o.iz + (dir / 9 - 1)) & mask;
                for (int32_t m = t.descend(o.level, x, y, z); t.nodes[m].level < o.level; m = t.descend(o.level, x, y, z)) {
                    t.split(m);
                    inner[t.nodes[m].level].push_back(m);
                }
            }
        }
    }
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

// For child c = (cz<<2)|(cy<<1)|cx of a node and direction dir: which neighbour of the node holds the child's neighbour
// octant, and as which of its children.
struct ChildStep { int8_t parent_dir, slot; };
struct ChildSteps {
    ChildStep at[8][kDirs];
    ChildSteps()
    {
        for (int c = 0; c < 8; ++c)
            for (int dir = 0; dir < kDirs; ++dir) {
                const int x = (c & 1) + dir % 3 - 1, y = ((c >> 1) & 1) + (dir / 3) % 3 - 1, z = (c >> 2) + dir / 9 - 1;   // -1 .. 2
                auto up = [](int p) { return p < 0 ? 0 : (p < 2 ? 1 : 2); };
                at[c][dir] = {static_cast<int8_t>(up(z) * 9 + up(y) * 3 + up(x)), static_cast<int8_t>(((z & 1) << 2) | ((y & 1) << 1) | (x & 1))};
            }
    }
};

// The children of an octant that touch the block on its side -dir: along an axis with d = -1 they are the upper
// children, with d = +1 the lower ones; axes with d = 0 are free and enumerated x, then y, then z (ascending Morton order).
struct TouchingChildren {
    int8_t count[kDirs], slot[kDirs][8];
    TouchingChildren()
    {
        for (int dir = 0; dir < kDirs; ++dir) {
            const int d[3] = {dir % 3 - 1, (dir / 3) % 3 - 1, dir / 9 - 1};
            int n = 0;
            for (int c = 0; c < 8; ++c) {
                bool touches = true;
                for (int ax = 0; ax < 3; ++ax)
                    if (d[ax] && ((c >> ax) & 1) != (d[ax] < 0 ? 1 : 0)) touches = false;
                if (touches) slot[dir][n++] = static_cast<int8_t>(c);
            }
            count[dir] = static_cast<int8_t>(n);
        }
    }
};

// The ghost table and what is derived from it: virtual blocks, and which parts of them are read.  The leaves have
// their ids.  Returns OT_OK or OT_E_UNBALANCED.
int make_tables(const Octree& t, HostTree& out)
{
    static const ChildSteps steps;
    static const TouchingChildren touching;
    const size_t nb = out.leaves.size();
    // neighbours of every node with children (the node itself in the middle), in the order of the nodes: parents come first
    std::vector<int32_t> rank(t.nodes.size(), -1), nbr;
    int32_t n_inner = 0;
    for (size_t n = 0; n < t.nodes.size(); ++n)
        if (t.nodes[n].first_child >= 0) rank[n] = n_inner++;
    nbr.assign(static_cast<size_t>(n_inner) * kDirs, 0);             // the root's neighbours are the root
    std::vector<int32_t> parent_of_leaf(nb, 0);                      // 8 * node + child
    for (size_t n = 0; n < t.nodes.size(); ++n) {
        if (t.nodes[n].first_child < 0) continue;
        const int32_t* at = &nbr[static_cast<size_t>(rank[n]) * kDirs];
        for (int c = 0; c < 8; ++c) {
            const int32_t ch = t.nodes[n].first_child + c;
            if (t.nodes[ch].first_child < 0) {
                parent_of_leaf[t.nodes[ch].leaf_id] = static_cast<int32_t>(8 * rank[n] + c);
                continue;
            }
            int32_t* to = &nbr[static_cast<size_t>(rank[ch]) * kDirs];
            for (int dir = 0; dir < kDirs; ++dir) {
                const ChildStep s = steps.at[c][dir];
                const int32_t first = t.nodes[at[s.parent_dir]].first_child;
                if (first < 0) return OT_E_UNBALANCED;
                to[dir] = first + s.slot;
            }
        }
    }
    // rows of the ghost table.  A neighbour octant under a leaf is that leaf's child octant: noted in `mask` (per leaf, which
    // of its child octants some block needs) and `coarser` (index of the entry, octant).
    std::vector<uint8_t> mask(nb, 0);
    struct Coarser { size_t entry; int32_t octant, dir; };
    std::vector<Coarser> coarser;
    out.ghost.clear();
    out.ghost.reserve(nb * kDirs * kEntry);
    for (size_t b = 0; b < nb; ++b) {
        const int c = parent_of_leaf[b] & 7;
        const int32_t* at = &nbr[static_cast<size_t>(parent_of_leaf[b] >> 3) * kDirs];
        int32_t row[kDirs * kEntry];
        for (int dir = 0; dir < kDirs; ++dir) {
            const ChildStep s = steps.at[c][dir];
            const Node& above = t.nodes[at[s.parent_dir]];
            int32_t* e = row + dir * kEntry;
            e[1] = e[2] = e[3] = e[4] = -1;
            if (above.first_child < 0) {
                e[0] = kCoarser;
                e[1] = above.leaf_id;
                mask[above.leaf_id] |= static_cast<uint8_t>(1 << s.slot);
                coarser.push_back({(b * kDirs + dir) * kEntry, s.slot, dir});
                continue;
            }
            const Node& nd = t.nodes[above.first_child + s.slot];
            if (nd.first_child < 0) {
                e[0] = kSame;
                e[1] = nd.leaf_id;
                continue;
            }
            e[0] = kFiner;
            for (int q = 0; q < touching.count[dir]; ++q) {
                const Node& ch = t.nodes[nd.first_child + touching.slot[dir][q]];
                if (ch.first_child >= 0) return OT_E_UNBALANCED;
                e[1 + q] = ch.leaf_id;
            }
        }
        out.ghost.insert(out.ghost.end(), row, row + kDirs * kEntry);
    }
    // virtual blocks, numbered by source leaf, then octant
    std::vector<int32_t> first(nb, 0);
    out.vblk.clear();
    int32_t n = 0;
    for (size_t s = 0; s < nb; ++s) {
        first[s] = n;
        for (int c = 0; c < 8; ++c)
            if ((mask[s] >> c) & 1) {
                out.vblk.push_back(static_cast<int32_t>(s));
                out.vblk.push_back(c);
                ++n;
            }
    }
    out.n_virt = n;
    out.ghost_v = out.ghost;
    out.vneed.assign(n, 0);
    // a block reads, of its neighbour in direction d, the three layers next to itself along every axis with d != 0
    // and all eight along the others
    auto layers = [](int d) { return d > 0 ? 0x07 : (d < 0 ? 0xE0 : 0xFF); };
    for (const Coarser& e : coarser) {
        int32_t* v = &out.ghost_v[e.entry];
        const int32_t src = v[1];
        v[0] = kVirtual;
        v[1] = first[src] + __builtin_popcount(static_cast<unsigned>(mask[src]) & ((1u << e.octant) - 1));
        out.vneed[v[1]] |= layers((e.dir / 3) % 3 - 1) | layers(e.dir / 9 - 1) << 8;
    }
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
    std::vector<int32_t> inner[21];
    // uniform refinement to lmin, then seed-driven refinement; each node is visited once
    while (!work.empty()) {
        const int32_t n = work.front();
        work.pop_front();
        const Node o = t.nodes[n];
        const bool grow = o.level < p.lmin || (o.level < p.lmax && near_seed(o, p));
        if (!grow) continue;
        inner[o.level].push_back(n);
        const int32_t first = t.split(n);
        for (int c = 0; c < 8; ++c) work.push_back(first + c);
    }
    balance(t, inner);
    out.leaves.clear();
    emit_leaves(t, 0, out.leaves);
    const int rc = make_tables(t, out);
    if (rc == OT_OK) make_units(out);
    return rc;
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
    out.leaves.clear();
    emit_leaves(t, 0, out.leaves);
    const int rc = make_tables(t, out);
    if (rc == OT_OK) make_units(out);
    return rc;
}

}  // namespace octfd
