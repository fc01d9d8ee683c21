// Where a ghost value of a block comes from, as 32 bits per value.  Private to the kernel files (and host code, so that
// the arithmetic can be checked on the CPU).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace octfd {
namespace {

constexpr int NPT = 8, PAD = 3, NP = 14, BLK = 512, PBLK = 2744;
constexpr int K_SAME = 0, K_FINER = 1, K_VIRT = 3;   // kinds of a ghost-table entry: copy, injection, copy from a virtual block

// A source is a byte offset into one variable's zipped array or array of virtual blocks.  Its three low bits are free:
// bit 0 says which of the two, bits 1 and 2 count the whole 4 GiB (2^20 blocks) that the offset leaves out.  The library
// refuses trees with 2^20 blocks or more, so these are 0 in the zipped array; but a coarse leaf has up to eight virtual
// blocks, and a sparsely refined tree has more than three times as many of them as blocks.
constexpr int64_t kBlockLimit = int64_t(1) << 20, kVirtualLimit = 4 * kBlockLimit;
constexpr int kBankShift = 20;                       // virtual block -> its 4 GiB

__host__ __device__ __forceinline__ bool source_is_virtual(uint32_t src) { return src & 1u; }
__host__ __device__ __forceinline__ uint64_t source_offset(uint32_t src) { return (uint64_t)((src >> 1) & 3u) << 32 | (src & ~7u); }

// the start, in doubles, of the 4 GiB that hold a virtual block
__host__ __device__ __forceinline__ int64_t bank_start(int32_t virtual_block) { return (int64_t)(virtual_block >> kBankShift) * BLK << kBankShift; }

// Where the point (lx, ly, lz) of the same-level octant in direction (rx, ry, rz) - 1 comes from, given that
// direction's entry e of the table in which coarser neighbours appear as virtual blocks: same level or virtual: copy;
// finer: the coinciding node of the child that holds it.
__host__ __device__ __forceinline__ uint32_t ghost_source(const int32_t* e, int rx, int ry, int rz, int lx, int ly, int lz)
{
    const int kind = e[0];
    uint32_t elem, low = 0;
    if (kind == K_SAME || kind == K_VIRT) {
        elem = (uint32_t)e[1] * BLK + (lz * NPT + ly) * NPT + lx;
        if (kind == K_VIRT) low = 1u | ((uint32_t)e[1] >> kBankShift) << 1;
    } else {
        // which child holds the point: forced by the direction on non-free axes
        const int bx = rx == 1 ? (lx >> 2) : (rx == 0 ? 1 : 0);
        const int by = ry == 1 ? (ly >> 2) : (ry == 0 ? 1 : 0);
        const int bz = rz == 1 ? (lz >> 2) : (rz == 0 ? 1 : 0);
        int q = 0, sh = 0;
        if (rx == 1) { q |= bx << sh; ++sh; }
        if (ry == 1) { q |= by << sh; ++sh; }
        if (rz == 1) { q |= bz << sh; }
        elem = (uint32_t)e[1 + q] * BLK + ((2 * lz - NPT * bz) * NPT + (2 * ly - NPT * by)) * NPT + (2 * lx - NPT * bx);
    }
    return elem * 8u | low;                          // modulo 2^32
}

}  // namespace
}  // namespace octfd
