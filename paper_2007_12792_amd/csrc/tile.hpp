// Global-memory access helpers and the workgroup -> block mapping.  Private to the kernel files (internal linkage throughout).
#pragma once
#include "kernels.hpp"
#include "lagrange.hpp"
#include "source.hpp"

namespace octfd {
namespace {

constexpr int NTHREADS = 512;

// Loads and stores of global arrays use a uniform 64-bit base (one variable's array) plus a 32-bit
// byte offset held per thread, so that no per-access 64-bit address arithmetic is needed.  The
// library refuses trees with 2^20 blocks or more, which keeps every offset into a zipped array below 2^32
// (for arrays of virtual blocks see source.hpp).
// The empty asm keeps the 32-bit offset a 32-bit register at the point of use; otherwise the
// compiler widens the offsets to 64 bits once, outside the variable loop, which doubles their
// register cost and forces a 64-bit add per access.
__device__ __forceinline__ double ldg(const double* base, uint32_t byte_off)
{
    asm volatile("" : "+v"(byte_off));
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + byte_off);
}
__device__ __forceinline__ void stg(double* base, uint32_t byte_off, double v)
{
    asm volatile("" : "+v"(byte_off));
    *reinterpret_cast<double*>(reinterpret_cast<char*>(base) + byte_off) = v;
}

// the value at a source, from the variable's zipped array or its virtual blocks
__device__ __forceinline__ double ldg_source(const double* base, const double* virt, uint32_t src)
{
    asm volatile("" : "+v"(src));
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(source_is_virtual(src) ? virt : base) + source_offset(src));
}

// NT: as non-temporal accesses, for data that would leave the caches before it is read again.
template <bool NT>
__device__ __forceinline__ double ldg(const double* base, uint32_t byte_off)
{
    if (!NT) return ldg(base, byte_off);
    asm volatile("" : "+v"(byte_off));
    return __builtin_nontemporal_load(reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + byte_off));
}
template <bool NT>
__device__ __forceinline__ void stg(double* base, uint32_t byte_off, double v)
{
    if (!NT) { stg(base, byte_off, v); return; }
    asm volatile("" : "+v"(byte_off));
    __builtin_nontemporal_store(v, reinterpret_cast<double*>(reinterpret_cast<char*>(base) + byte_off));
}

// two neighbouring values; arrays are only known to be aligned to 8 bytes, which 16-byte accesses allow
typedef double Pair __attribute__((ext_vector_type(2)));
typedef Pair PairAt8 __attribute__((aligned(8)));

// Workgroups are handed to the eight XCDs (each with its own L2) round-robin by workgroup id.
// Chunks of 16 Morton-consecutive blocks (two sibling octets) are dealt to the XCDs in turn: blocks
// that run at the same time on one XCD are then close neighbours, which read each other's rows
// through the same L2, while every XCD still sees the same mix of cheap and expensive blocks.
// (Measured on the 102,075-block tree: 78.0 ms per step against 83.5 ms with one contiguous eighth
// of the Morton order per XCD and 78.4 ms with no remapping.)
constexpr int NXCD = kSchedXcds;
template <int XCD_CHUNK = kSchedChunk>
__device__ __forceinline__ int64_t block_of_workgroup(int64_t wg)
{
    const int64_t x = wg % NXCD, q = wg / NXCD;
    return (q / XCD_CHUNK) * (XCD_CHUNK * NXCD) + x * XCD_CHUNK + (q % XCD_CHUNK);   // may be >= nb: caller checks
}
template <int XCD_CHUNK = kSchedChunk>
inline unsigned grid_for_blocks(int64_t nb)
{
    const int64_t span = XCD_CHUNK * NXCD;
    return (unsigned)((nb + span - 1) / span * span);
}

}  // namespace
}  // namespace octfd
