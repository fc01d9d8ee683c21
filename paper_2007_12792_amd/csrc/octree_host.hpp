// Host-side octree engine of liboctfd: pointer octree, 2:1 balance, Morton-order
// traversal and the ghost-source table.  No device code here.
#pragma once
#include <cstdint>
#include <cstdlib>
#include <new>
#include <vector>

#include <sys/mman.h>

#include "octfd.h"

namespace octfd {

constexpr int kDirs = 27;          // directions (dz+1)*9 + (dy+1)*3 + (dx+1)
constexpr int kEntry = 5;          // {kind, id0..id3}
enum GhostKind : int32_t { kSame = 0, kFiner = 1, kCoarser = 2, kVirtual = 3 };

// Allocator of the two big tables (540 bytes per block each): whole huge pages where the system gives them on request.
// A fresh table is written once, and with pages of 4 KB the page faults took longer than everything else in building a
// tree (26 of 27 ms for 27,756 blocks on a virtual machine; 12 of 18 with huge pages).
template <class T>
struct HugePageAllocator {
    using value_type = T;
    static constexpr size_t kPage = size_t(2) << 20;
    HugePageAllocator() = default;
    template <class U> HugePageAllocator(const HugePageAllocator<U>&) {}
    T* allocate(size_t n)
    {
        if (n > (~size_t(0) - kPage) / sizeof(T)) throw std::bad_alloc();
        size_t bytes = n * sizeof(T);
        const bool huge = bytes >= kPage;
        if (huge) bytes = (bytes + kPage - 1) / kPage * kPage;
        void* p = huge ? std::aligned_alloc(kPage, bytes) : std::malloc(bytes ? bytes : 1);
        if (!p) throw std::bad_alloc();
        if (huge) (void)madvise(p, bytes, MADV_HUGEPAGE);            // a hint: without it the pages are small ones
        return static_cast<T*>(p);
    }
    void deallocate(T* p, size_t) { std::free(p); }
    template <class U> bool operator==(const HugePageAllocator<U>&) const { return true; }
    template <class U> bool operator!=(const HugePageAllocator<U>&) const { return false; }
};
using BigTable = std::vector<int32_t, HugePageAllocator<int32_t>>;

struct HostTree {
    std::vector<ot_leaf> leaves;   // Morton order
    BigTable ghost;                // [nb][27][5]
    // "Virtual blocks".  Where the same-level neighbour octant of a block does not exist because its parent L is
    // a leaf, the ghost values in that direction are interpolated inside L, and what they are depends only on L's
    // data and on the fine position inside L, not on which block asks.  Such an octant can therefore be filled
    // once, like a child of L ("virtual block"), after which the blocks around it read it
    // exactly like a neighbour of their own level.
    //   vblk    [n_virt][2]        per virtual block {source leaf id, child octant (ox | oy<<1 | oz<<2)}, ordered by
    //                              source leaf (Morton order), then octant
    //   ghost_v [nb][27][5]        the ghost table with every coarser entry replaced by {kVirtual, virtual block}
    //   n_virt                     number of virtual blocks
    //   vneed   [n_virt]           which y rows (bits 0..7) and z planes (bits 8..15) of a virtual block any block reads: the
    //                              union, per axis, over the blocks that have it as a neighbour.  The fill writes only
    //                              those (whole x rows of them); the rest of a virtual block is never read.
    BigTable ghost_v;
    std::vector<int32_t> vblk, vneed;
    int64_t n_virt = 0;
    // Work units of the two-block kernel of the 24-field system, in Morton order: the first block of every two
    // leaves that are the lower and upper x child of one parent (they follow each other in storage), and, flagged
    // with kUnitSingle, every other block (a leaf whose x sibling is subdivided).  Every block belongs to exactly one unit.
    std::vector<int32_t> units;
};

// Each returns an OT_* status.
int build_tree(const ot_build_params& p, HostTree& out);
int tree_from_leaves(const ot_leaf* leaves, size_t n, HostTree& out);
void make_units(HostTree& t);

}  // namespace octfd
