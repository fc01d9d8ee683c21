// LDS tile of one block and one variable: geometry, per-block table rows, the order in which the
// tile is filled ("fill plan"), global-memory access helpers and the workgroup -> block mapping.
// Private to kernels.hip (internal linkage throughout).
#pragma once
#include "kernels.hpp"
#include "lagrange.hpp"
#include "source.hpp"

namespace octfd {
namespace {

constexpr int NTHREADS = 512;

// LDS geometry (in doubles).  Rows are stored compactly (stride 14) and planes are padded to a
// stride of 200 = 8 (mod 32).  A wavefront holds one j row of the block, its lanes run over
// (i, k): the eight x-contiguous values of four consecutive k planes then fall into 32 different
// 8-byte banks, and shifting the access by any stencil offset keeps that property.
// wavefronts per SIMD the right-hand-side kernels are compiled for: the 24-field kernel 4 (128 VGPRs per lane, two
// workgroups share a compute unit, which is also what its LDS allows); the other kinds 8 (64 VGPRs, four workgroups)
constexpr int waves_per_simd(int kind) { return kind == OT_RHS_SYN24 ? 4 : 8; }
constexpr int RS = NP;                   // 14
constexpr int PS = NP * RS + 4;          // 200
constexpr int TILE = NP * PS;            // 14 planes
constexpr int WZ = NPT * PS;             // D1_z u on [8 k][14 jj][14 ii]
constexpr int YPS = NPT * RS + 8;        // plane stride of the D1_y array, 120 = 24 (mod 32)
constexpr int WY = NPT * YPS;            // D1_y u on [8 k][8 j][14 ii]

__device__ __forceinline__ int tidx(int kk, int jj, int ii) { return kk * PS + jj * RS + ii; }

// thread -> interior point: lanes run over (i, k), the wavefront number is j.
__device__ __forceinline__ void point_of(int tid, int& i, int& j, int& k)
{
    i = tid & 7;
    k = (tid >> 3) & 7;
    j = tid >> 6;
}

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

// the value at a source, from the variable's zipped array or its virtual blocks; WIDE = false: of a tree with at most
// kBlockLimit virtual blocks, whose bits 1 and 2 are 0
template <bool WIDE = true>
__device__ __forceinline__ double ldg_source(const double* base, const double* virt, uint32_t src)
{
    if (!WIDE) return ldg(source_is_virtual(src) ? virt : base, src & ~1u);
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

// ---------------------------------------------------------------- fill plan

// The 2,744 points of the tile are enumerated so that a prefix of the enumeration is exactly what a
// kernel needs:
//   [0, NFACE)      interior and the six face slabs: all that stencils along the axes read;
//   [NFACE, NEDGE)  the twelve edge slabs: read in addition by the mixed second derivatives;
//   [NEDGE, PBLK)   the eight corners: needed only when the whole padded block is written out.
// Fetching only the prefix in use matters because every 8-point ghost row is a 64-byte half of a
// 128-byte line of the neighbour's zipped storage, of which an x ghost uses three values: faces
// alone touch 288 rows per tile (152 lines), faces and edges 516 rows (288 lines), the full tile
// 588 rows (336 lines).
constexpr int NFACE = BLK + 6 * PAD * NPT * NPT;                 // 1664
constexpr int NEDGE = NFACE + 12 * PAD * PAD * NPT;              // 2528
constexpr int PLAN_FACE = (NFACE + NTHREADS - 1) / NTHREADS;     // 4 entries per thread
constexpr int PLAN_EDGE = (NEDGE + NTHREADS - 1) / NTHREADS;     // 5

__device__ __forceinline__ int ghost_index(int g) { return g < PAD ? g : g + NPT; }   // 0,1,2,11,12,13

__device__ __forceinline__ void tile_point(int p, int& ii, int& jj, int& kk)
{
    if (p < 14 * 64) {                               // x-extended interior rows
        const int r = p / NP;
        ii = p - r * NP; jj = PAD + (r & 7); kk = PAD + (r >> 3);
    } else if (p < 14 * 64 + 384) {                  // y faces
        const int q = p - 14 * 64, r = q >> 3, kq = r / 6;
        ii = PAD + (q & 7); jj = ghost_index(r - 6 * kq); kk = PAD + kq;
    } else if (p < NFACE) {                          // z faces
        const int q = p - (14 * 64 + 384);
        ii = PAD + (q & 7); jj = PAD + ((q >> 3) & 7); kk = ghost_index(q >> 6);
    } else if (p < NFACE + 288) {                    // xy edges
        const int q = p - NFACE, r = q / 6, kq = r / 6;
        ii = ghost_index(q - 6 * r); jj = ghost_index(r - 6 * kq); kk = PAD + kq;
    } else if (p < NFACE + 576) {                    // xz edges
        const int q = p - (NFACE + 288), r = q / 6;
        ii = ghost_index(q - 6 * r); jj = PAD + (r & 7); kk = ghost_index(r >> 3);
    } else if (p < NEDGE) {                          // yz edges
        const int q = p - (NFACE + 576), r = q >> 3, kq = r / 6;
        ii = PAD + (q & 7); jj = ghost_index(r - 6 * kq); kk = ghost_index(kq);
    } else {                                         // corners
        const int q = p - NEDGE, r = q / 6, kq = r / 6;
        ii = ghost_index(q - 6 * r); jj = ghost_index(r - 6 * kq); kk = ghost_index(kq);
    }
}

// Entries with nothing to copy (beyond the range in use, or interpolated later) read element 0 and
// write to DUMMY, a padding slot of the tile that no stencil reads; the copy loop is branch-free.
constexpr int DUMMY = NP * RS;   // first padding slot behind plane 0
// src: byte offset in the source array, needed once per variable and kept in LDS as src[m * NTHREADS + tid];
// dst: tile index, two 16-bit values per register.
template <int NPLAN>
struct FillPlan {
    uint32_t* src;
    uint32_t dstp[(NPLAN + 1) / 2];
    __device__ __forceinline__ int dst(int m) const { return (dstp[m >> 1] >> (16 * (m & 1))) & 0xffff; }
    __device__ __forceinline__ void set_dst(int m, int v) { dstp[m >> 1] = (m & 1) ? (dstp[m >> 1] | ((uint32_t)v << 16)) : (uint32_t)v; }
};
static_assert(TILE < 65536, "tile indices are packed in pairs");

// Source of every padded point this thread fills, as a byte offset into the block's padded data.
// NPOINTS = how long a prefix of the enumeration is planned.
template <int NPLAN, int NPOINTS>
__device__ __forceinline__ void make_plan_padded(FillPlan<NPLAN>& fp, int tid)
{
#pragma unroll
    for (int m = 0; m < NPLAN; ++m) {
        const int p = tid + m * NTHREADS;
        const bool ok = p < NPOINTS;
        int ii, jj, kk;
        tile_point(ok ? p : 0, ii, jj, kk);
        fp.src[m * NTHREADS + tid] = ok ? (uint32_t)((kk * NP + jj) * NP + ii) * 8u : 0u;
        fp.set_dst(m, ok ? tidx(kk, jj, ii) : DUMMY);
    }
}

}  // namespace
}  // namespace octfd
