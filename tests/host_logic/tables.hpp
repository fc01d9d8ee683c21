// The ghost table of a tree in full, [nb][27][5], for the host-only checks: as the library hands it out, and as the device makes it for
// itself, coarser neighbours as virtual blocks.
#pragma once
#include <vector>

#include "octree_host.hpp"

inline std::vector<int32_t> ghost_table(const octfd::HostTree& t)
{
    std::vector<int32_t> out(t.leaves.size() * octfd::kDirs * octfd::kEntry);
    octfd::write_ghost_table(t, out.data());
    return out;
}

inline std::vector<int32_t> ghost_table_by_entry(const octfd::HostTree& t, bool virt)
{
    std::vector<int32_t> out;
    out.reserve(t.leaves.size() * octfd::kDirs * octfd::kEntry);
    int32_t e[octfd::kEntry];
    for (size_t b = 0; b < t.leaves.size(); ++b)
        for (int dir = 0; dir < octfd::kDirs; ++dir) {
            octfd::table_entry(t.source(), static_cast<int64_t>(b), dir, virt, e);
            out.insert(out.end(), e, e + octfd::kEntry);
        }
    return out;
}
