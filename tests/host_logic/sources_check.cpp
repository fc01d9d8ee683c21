// Host-only check of the 32-bit sources of ghost values (csrc/source.hpp) on a tree with more than 2^20 virtual blocks: every
// entry of the table, at the corners of the octant, against the index worked out in 64 bits.  Built with g++ together with
// csrc/octree_host.cpp by tests/test_many_virtual_blocks.py.
#include <cstdio>
#include <vector>

#include "octree_host.hpp"
#include "source.hpp"
#include "tables.hpp"

using namespace octfd;

int main()
{
    // level 6 for z < 40 of 64, level 5 above; of the level-6 octants with even coordinates those with z = 2 .. 38 are split
    std::vector<ot_leaf> lv;
    for (uint32_t z = 0; z < 40; ++z)
        for (uint32_t y = 0; y < 64; ++y)
            for (uint32_t x = 0; x < 64; ++x) {
                if ((x | y | z) & 1 || z < 2) { lv.push_back({6, x, y, z}); continue; }
                for (uint32_t c = 0; c < 8; ++c) lv.push_back({7, 2 * x + (c & 1), 2 * y + ((c >> 1) & 1), 2 * z + (c >> 2)});
            }
    for (uint32_t z = 20; z < 32; ++z)
        for (uint32_t y = 0; y < 32; ++y)
            for (uint32_t x = 0; x < 32; ++x) lv.push_back({5, x, y, z});
    HostTree t;
    if (tree_from_leaves(lv.data(), lv.size(), t) != OT_OK) { std::printf("FAILED: tree\n"); return 1; }
    const long nb = static_cast<long>(t.leaves.size());
    std::printf("blocks %ld, virtual blocks %ld\n", nb, static_cast<long>(t.n_virt));
    if (t.n_virt <= kBlockLimit || nb >= kBlockLimit || t.n_virt > kVirtualLimit) { std::printf("FAILED: sizes\n"); return 1; }
    const std::vector<int32_t> ghost_v = ghost_table_by_entry(t, true);
    long bad = 0, beyond = 0;
    for (long b = 0; b < nb; ++b)
        for (int dir = 0; dir < kDirs; ++dir) {
            const int32_t* e = &ghost_v[(b * kDirs + dir) * kEntry];
            const int r[3] = {dir % 3, (dir / 3) % 3, dir / 9};
            for (int corner = 0; corner < 8; ++corner) {
                const int l[3] = {corner & 1 ? 7 : 0, corner & 2 ? 7 : 0, corner & 4 ? 7 : 0};
                int64_t block = e[1], point = (l[2] * NPT + l[1]) * NPT + l[0];
                if (e[0] == kFiner) {                // the child that holds the point, its coinciding node
                    // only the children next to the block exist in the entry: those on the near side along directed axes
                    bool near_side = true;
                    for (int ax = 0; ax < 3; ++ax)
                        if (r[ax] != 1 && (l[ax] > 3) != (r[ax] == 0)) near_side = false;
                    if (!near_side) continue;
                    int q = 0, sh = 0;
                    for (int ax = 0; ax < 3; ++ax)
                        if (r[ax] == 1) q |= (l[ax] > 3) << sh++;
                    block = e[1 + q];
                    point = ((2 * l[2] & 7) * NPT + (2 * l[1] & 7)) * NPT + (2 * l[0] & 7);
                }
                const uint32_t s = ghost_source(e, r[0], r[1], r[2], l[0], l[1], l[2]);
                const uint64_t want = static_cast<uint64_t>(block * BLK + point) * 8;
                beyond += want >> 32 != 0;
                bad += source_offset(s) != want || source_is_virtual(s) != (e[0] == kVirtual);
                if (e[0] == kVirtual)                // a face's base and offset, as the slab kernels take them
                    bad += static_cast<uint64_t>(bank_start(e[1])) * 8 + static_cast<uint32_t>((static_cast<uint32_t>(e[1]) * BLK + point) * 8u) != want;
            }
        }
    std::printf("offsets beyond 2^32: %ld, wrong: %ld\n", beyond, bad);
    if (bad || !beyond) { std::printf("FAILED: sources\n"); return 1; }
    return 0;
}
