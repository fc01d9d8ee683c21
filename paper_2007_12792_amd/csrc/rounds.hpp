// How the 24-field kernel with two points per thread (brick.hip) deals the units of a tree to its workgroups.  Private to the kernel
// files (and host code, so that the dealing can be checked on the CPU).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"

namespace octfd {
namespace {

// A workgroup fills a compute unit.  Round r is units 256 r .. 256 r + 255, one per compute unit, of which each XCD (workgroup i runs on
// XCD i mod 8) takes a run, so that the blocks it works on at a time are close neighbours.  -1: none for workgroup `wg` in this round.
constexpr int kRound = 256;
__host__ __device__ __forceinline__ int64_t unit_of_round(int64_t round, int wg, int64_t n_units)
{
    const int64_t left = n_units - round * kRound;
    if (left <= 0) return -1;
    const int run = left < kRound ? (int)((left + kSchedXcds - 1) / kSchedXcds) : kRound / kSchedXcds;   // the last round is spread over all XCDs
    const int x = wg % kSchedXcds, n = wg / kSchedXcds;
    return n < run && x * run + n < left ? round * kRound + x * run + n : -1;
}
__host__ __device__ __forceinline__ int64_t rounds_of(int64_t n_units) { return (n_units + kRound - 1) / kRound; }

// A launch is that many parts of 256 workgroups, each for half of the rounds that are left, the last one for the rest; a workgroup goes through
// the rounds of its part.  Where another stream's kernel holds a compute unit, one of the first 256 workgroups starts when the
// others end, and the workgroups of the later parts go to whichever compute unit is free.  Two rounds are not divided: the last workgroups
// of an XCD have one unit less than the first.  (us a step, on its own / while another kernel holds one compute unit of each XCD, one part -> as
// here: 1,541 blocks 901 / 1076 -> 904 / 875, 3,067 1649 / 2130 -> 1657 / 1708, 21,057 9433 / 14,457 -> 9465 / 10,079, 102,040 43,097 / 68,871 -> 43,067 /
// 47,098; 1,016 blocks, two rounds, 639 / 734.  Equal parts of eight rounds, 21,057 blocks: 9488 / 10,237.  Evaluations on padded blocks gain a
// hundredth by themselves: 21,057 blocks 3448 -> 3408.)
constexpr int kMostParts = 6;
inline int parts_of(int64_t rounds)
{
    int parts = 1;
    while (parts < kMostParts && rounds > int64_t(1) << parts) ++parts;
    return parts;
}
struct Rounds { int64_t first, last; };
__host__ __device__ __forceinline__ Rounds rounds_of_part(int part, int parts, int64_t rounds)
{
    return {rounds - (rounds >> part), part == parts - 1 ? rounds : rounds - (rounds >> (part + 1))};
}

}  // namespace
}  // namespace octfd
