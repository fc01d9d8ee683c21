// gfx950 kernels of liboctfd.
//
// A workgroup owns one block.  The kinds with one or two variables read it in slabs of two planes, one per wavefront
// (slab.hpp); the 24-field system has kernels of its own (brick.hip, pair.hip).  The fused kernels take ghost
// values straight from zipped storage through the ghost-source table and never materialise the padded array.
//
// Arithmetic follows one fixed IEEE sequence per formula (see octfd.h); the file is compiled with
// -ffp-contract=off, so a fused multiply-add happens exactly where fma() is written.
#include "slab.hpp"
#include "stencils.hpp"
#include "tile.hpp"

#include <algorithm>
#include <type_traits>

namespace octfd {
namespace {

// ---------------------------------------------------------------- right-hand-side kernel

// The right-hand side (and Runge-Kutta stage update) of whole blocks, one block per workgroup, all its variables.
// Zipped input (ZIN): the block's surroundings are read through the ghost table in which coarser neighbours appear as
// virtual blocks, which k_virtual or k_virtual_centred has filled before the launch, so every value is a copy or an
// injection and no interpolation happens here; the two ghost rules differ only in which of the two kernels ran.
constexpr int rhs_threads(int kind) { return slab_wavefronts(kind) * 64; }
constexpr int kWavesPerSimd = 8;                     // 64 VGPRs: four workgroups share a compute unit
template <int KIND, bool ZIN, int EPI>
__global__ __launch_bounds__(rhs_threads(KIND), kWavesPerSimd) void k_rhs(DeviceTree tr, RhsArgs a)
{
    static_assert(ZIN != (EPI == kOutPadded), "padded in, padded out; everything else zipped");
    const int64_t b = block_of_workgroup(blockIdx.x);
    if (b >= tr.nb) return;                          // uniform over the workgroup
    __shared__ double lds[slab_wavefronts(KIND) / sl::NSLAB * sl::LDS];
    __shared__ double lapS[KIND == OT_RHS_WAVE ? BLK : 1];
    rhs_slab<KIND, ZIN, EPI, false>(tr, a, lds, lapS, b, threadIdx.x);
}
// The same on zipped input with non-temporal accesses to everything but the input (see streams()): what passes through once
// does not push the input, whose ghost rows are read by several blocks, out of the L2 and the memory-side cache.
constexpr int kStreamChunk = 64;   // blocks dealt to an XCD at a time: 1541 / 1521 / 1515 / 1509 / 1535 us for 8 / 16 / 32 / 64 / 128
                                   // (step of the wave system on 47,783 blocks)
template <int KIND, int EPI>
__global__ __launch_bounds__(rhs_threads(KIND), kWavesPerSimd) void k_rhs_stream(DeviceTree tr, RhsArgs a)
{
    const int64_t b = block_of_workgroup<kStreamChunk>(blockIdx.x);
    if (b >= tr.nb) return;
    __shared__ double lds[slab_wavefronts(KIND) / sl::NSLAB * sl::LDS];
    __shared__ double lapS[KIND == OT_RHS_WAVE ? BLK : 1];
    rhs_slab<KIND, true, EPI, true>(tr, a, lds, lapS, b, threadIdx.x);
}

// padded blocks in and out, written non-temporally (see kStreamPaddedBytes; an instance of its own, since a branch around the two kinds of
// store is merged into one plain store)
template <int KIND>
__global__ __launch_bounds__(rhs_threads(KIND), kWavesPerSimd) void k_rhs_padded_stream(DeviceTree tr, RhsArgs a)
{
    const int64_t b = block_of_workgroup(blockIdx.x);
    if (b >= tr.nb) return;
    __shared__ double lds[slab_wavefronts(KIND) / sl::NSLAB * sl::LDS];
    __shared__ double lapS[KIND == OT_RHS_WAVE ? BLK : 1];
    rhs_slab<KIND, false, kOutPadded, true>(tr, a, lds, lapS, b, threadIdx.x);
}

// ---------------------------------------------------------------- unzip / zip kernels

// unzip as a gather.  With the virtual blocks of the input filled (by k_virtual for the clamped ghost rule, by
// k_virtual_centred for the centred one), every one of the 2,744 points of a padded block is a copy: of the block's
// own data, of a same-level or virtual neighbour, or of the coinciding node of a finer neighbour.
// What bounds it is the output (5.4 times the input) together with the reads of ghost rows, of which an x ghost uses three
// values of eight.  A wavefront reads the rows of one plane in groups that lie in whole 128-byte lines of their sources:
// three rows below the block, four and four of it, three above, so that no line is asked for by two wavefronts at a time
// (the L1 stalls on a request for a line that is still on its way).  The values meet in LDS, from where they leave in
// whole lines, 16 bytes a lane; the sources are kept in registers for all variables of the workgroup, and the
// loads of the next variable are in flight while one is written.  The stores are non-temporal: the padded output is not
// read again here and would otherwise push the ghost rows out of the L2.
// A workgroup takes every `stride`-th variable of a block.  Normally that is all of them, chunks of 16 consecutive blocks
// dealt to the XCDs in turn; on small trees the variables are split so that the chip is full (unzip_stride).
// (21,064 blocks, 24 variables: 4.24 -> 3.68 ms; 47,783 blocks, two variables: 807 -> 664 us.  Before, a thread copied six
// points 512 apart from memory to memory, eight workgroups per block, one variable of eight each.  Chunks of
// 8 / 64 / 128 blocks: 3.71 / 3.71 / 3.79 ms; plain stores +8 %; two buffers in LDS with one barrier per variable +1 to 7 %.
// Where the output stays in the memory-side cache, the call by itself is slower than that with four variables or more: 24
// on 512 blocks 52 -> 61 us, 8 on 1,513 blocks 69 -> 78, 4 on 3,004 76 -> 79.  The launch that reads the output gains more:
// unzip, rhs_eval and zip of the 24-field system 241 -> 225 us on 512 blocks, 420 -> 404 on 820, 757 -> 715 on 1,513.)
// Workgroups per block: 1,024 run at a time, and four times as many keep the last wave short; but at least two variables each,
// for which the sources are worked out once (792 blocks, 24 variables, 1 / 2 / 6 / 12 per block: 167 / 161 / 154 / 157 us; 834
// blocks, two variables, 1 / 2 per block: 12.4 / 14.2 us).
inline int unzip_stride(int64_t nb, int nvar) { return (int)std::max<int64_t>(1, std::min<int64_t>(nvar / 2, (4096 + nb - 1) / nb)); }
constexpr int kUnzipRows = NP * 4 / (NTHREADS / 64);   // row groups per wavefront: 7
__global__ __launch_bounds__(NTHREADS, 8) void k_unzip(DeviceTree tr, int nvar, int stride, const double* __restrict__ zipped,
                                                       const double* __restrict__ virt, double* __restrict__ padded)
{
    __shared__ int32_t gt[27 * 5];
    __shared__ __attribute__((aligned(16))) double T[PBLK];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int64_t b = block_of_workgroup(blockIdx.x), nb = tr.nb;
    const int v0 = (int)blockIdx.y;
    if (b >= nb) return;                             // uniform over the workgroup
    if (tid < 27 * 5) gt[tid] = tr.ghost_v[b * (27 * 5) + tid];
    __syncthreads();
    // the wavefront's row group: rows 0..2, 3..6, 7..10 or 11..13 of the planes wave / 4, + 2, + 4, ...
    const int group = wave & 3, row0 = group * 4 - (group > 0 ? 1 : 0), rows = group == 0 || group == 3 ? PAD : 4;
    const bool mine = lane < rows * NP;
    const int row = min(lane / NP, rows - 1), ii = lane % NP, jj = row0 + row;
    const int rx = ii < PAD ? 0 : (ii < PAD + NPT ? 1 : 2), ry = group == 0 ? 0 : (group == 3 ? 2 : 1);
    const int lx = ii - PAD + (1 - rx) * NPT, ly = jj - PAD + (1 - ry) * NPT;
    uint32_t off[kUnzipRows];
#pragma unroll
    for (int m = 0; m < kUnzipRows; ++m) {
        const int kk = (wave >> 2) + 2 * m;
        const int rz = kk < PAD ? 0 : (kk < PAD + NPT ? 1 : 2), lz = kk - PAD + (1 - rz) * NPT;
        off[m] = ghost_source(&gt[(rz * 9 + ry * 3 + rx) * 5], rx, ry, rz, lx, ly, lz);   // the centre entry is the block itself
    }
    double pv[kUnzipRows];
    auto load = [&](int v) {
        const double* base = zipped + (int64_t)v * nb * BLK;
        const double* vbase = virt + (int64_t)v * tr.n_virt * BLK;
        if (mine) {
#pragma unroll
            for (int m = 0; m < kUnzipRows; ++m) pv[m] = ldg_source(base, vbase, off[m]);
        }
    };
    double* const t = T + (wave >> 2) * (NP * NP) + row0 * NP + lane;
    load(v0);
#pragma unroll 1
    for (int v = v0; v < nvar; v += stride) {
        if (mine) {
#pragma unroll
            for (int m = 0; m < kUnzipRows; ++m) t[2 * m * (NP * NP)] = pv[m];
        }
        __syncthreads();
        if (v + stride < nvar) load(v + stride);
        // blocks are 171.5 lines long: every second one starts in the middle of a line
        const int64_t q = (int64_t)v * nb + b;
        PairAt8* out = reinterpret_cast<PairAt8*>(padded + q * PBLK);
        const int first = tid - ((q & 1) ? 4 : 0);
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int n = first + m * NTHREADS;
            if (n >= 0 && n < PBLK / 2) __builtin_nontemporal_store(reinterpret_cast<const Pair*>(T)[n], out + n);
        }
        __syncthreads();                                         // the next variable overwrites the array
    }
}

// Virtual blocks.  A virtual block is a child octant o of its source leaf; its 8^3 points are the fine positions
// f = 8 o + i per axis inside the leaf, interpolated x, then y, then z like any ghost point that comes from a
// coarser leaf.  Here a LANE owns a whole line of a pass: it holds the line's eight coarse nodes in registers and
// produces its eight fine values (four pass through, four take the clamped six-point stencil; which ones is the
// same for all lanes, so the weights are constants).  A wavefront owns one variable of the block: its 64 lanes are
// the 64 lines of a pass, the passes hand over through a staging array of the wavefront's own, in place, and nothing
// needs a workgroup barrier.  The eight wavefronts of a workgroup take eight variables of one virtual block at a time
// (or, with fewer variables, of several virtual blocks).
// (The same passes with one thread per point were bound by LDS instructions: 1.3 ms per call on the 102,075-block tree.)

// the eight fine values r of a child half (O = 0 lower, 1 upper) of a line with nodes v: for odd f = 8 O + i the same
// sequence as interp_line (first node s = clamp(c0 - 2, 0, 2), c0 = (f - 1) / 2; acc = w0 v_s, then five fma)
template <int O>
__device__ __forceinline__ void fine_half_line(const double (&v)[8], double (&r)[8])
{
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        r[2 * n] = v[4 * O + n];
        constexpr int kLo = 0;
        const int c0 = 4 * O + n, s = c0 - 2 < kLo ? kLo : (c0 - 2 > 2 ? 2 : c0 - 2), row = c0 - s;
        double acc = c_lag[row * 6] * v[s];
#pragma unroll
        for (int m = 1; m < 6; ++m) acc = fma(c_lag[row * 6 + m], v[s + m], acc);
        r[2 * n + 1] = acc;
    }
}
__device__ __forceinline__ void fine_line(int o, const double (&v)[8], double (&r)[8])
{
    if (o) fine_half_line<1>(v, r);                  // uniform
    else fine_half_line<0>(v, r);
}

// From this size of the input on the fills write non-temporally: the virtual blocks are read once or twice, among data many times the
// memory-side cache.  (us, plain / non-temporal, step, step with the centred rule, evaluation, unzip: 24 fields on 3,396 blocks, 334 MB, 1711 / 1687,
// 1894 / 1876, 345 / 333, 695 / 690, on 21,064 9566 / 9444, 10380 / 10270, 1899 / 1876, 4078 / 4040; wave system on 47,783, 391 MB, 1503 / 1491,
// 1595 / 1593, 261 / 258, 728 / 724.  Below: 24 fields on 1,919, 188 MB, 978 / 980, 1083 / 1088, 188 / 180, 379 / 382; wave system on 21,064,
// 173 MB, 684 / 681, 752 / 752, 102 / 106, 251 / 290; Burgers on 47,783, 196 MB, 694 / 693, 751 / 750, 111 / 105, 351 / 337, on 21,064 unzip 123 / 150.  Just
// above, on trees with 1.0, 0.45 and 0.36 virtual blocks per block: 24 fields 259 MB 1424 / 1409, 1600 / 1590, 290 / 284, 549 / 542, 289 MB 1493 / 1470, 1657 / 1642,
// 293 / 291, 608 / 602; wave 259 MB 1010 / 1007, 1084 / 1085, 175 / 172, 482 / 480, 290 MB 1114 / 1110, 1189 / 1189, 192 / 192, 531 / 530; Burgers 259 MB 913 /
// 912, 977 / 977, 150 / 149, 483 / 482, 289 MB 1015 / 1016, 1082 / 1084, 165 / 164, 538 / 534.)
constexpr int64_t kStreamFillBytes = 256ll << 20;
inline bool fill_streams(const DeviceTree& t, int nvar) { return nvar * t.nb * BLK * (int64_t)sizeof(double) > kStreamFillBytes; }
template <bool NT>
__device__ __forceinline__ void put_virtual(double* p, double v)
{
    if (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}
constexpr int VPS = 72;                              // plane stride of the staging array, 8 (mod 32): no bank conflicts in the y pass
template <bool NT>
__global__ __launch_bounds__(NTHREADS) void k_virtual(DeviceTree tr, int nvar, const double* __restrict__ zipped, double* __restrict__ virt)
{
    __shared__ double staging[8][NPT * VPS];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // with fewer than eight variables a workgroup takes several virtual blocks, so that no wavefront idles:
    // wavefront w -> virtual block `sub` of the workgroup's `per`, variables v0, v0 + nv, ...
    const int nv = nvar < 8 ? nvar : 8, per = 8 / nv;
    const int sub = wave / nv, v0 = wave - sub * nv;
    // runs of 16 consecutive workgroups (the children of a few source leaves) go to one XCD, whose L2 then serves
    // the re-reads of a source leaf by its other children
    const int64_t q = block_of_workgroup(blockIdx.x) * per + sub, nb = tr.nb;
    if (sub >= per || q >= tr.n_virt) return;        // uniform over the wavefront; the kernel has no workgroup barrier
    const int64_t leaf = tr.vblk[2 * q];
    const int oct = tr.vblk[2 * q + 1];
    const int need = tr.vneed[q];                                // y rows and z planes that any block reads
    const int ox = oct & 1, oy = (oct >> 1) & 1, oz = oct >> 2;
    const int hi = lane >> 3, lo = lane & 7;
    const bool row_needed = (need >> hi) & 1;
    double* A = staging[wave];
    const int64_t in_stride = nb * BLK, out_stride = tr.n_virt * BLK;
    const double* in = zipped + leaf * BLK + lane * NPT;        // x pass: this lane's line is (cz, cy) = (hi, lo)
    double* out = virt + q * BLK + lane;                        // z pass: this lane's line is (ty, tx) = (hi, lo)
    double nxt[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) nxt[m] = in[v0 * in_stride + m];
#pragma unroll 1
    for (int v = v0; v < nvar; v += nv) {
        double c[8], r[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) c[m] = nxt[m];
        if (v + nv < nvar) {
#pragma unroll
            for (int m = 0; m < 8; ++m) nxt[m] = in[(v + nv) * in_stride + m];
        }
        fine_line(ox, c, r);                                    // (cz, cy) -> fine x
#pragma unroll
        for (int m = 0; m < 8; ++m) A[hi * VPS + lo * NPT + m] = r[m];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int m = 0; m < 8; ++m) c[m] = A[hi * VPS + m * NPT + lo];      // line (cz, tx) = (hi, lo) over cy
        fine_line(oy, c, r);
        // in place: a lane writes exactly the positions it has just read
#pragma unroll
        for (int m = 0; m < 8; ++m) A[hi * VPS + m * NPT + lo] = r[m];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int m = 0; m < 8; ++m) c[m] = A[m * VPS + lane];              // line (ty, tx) = (hi, lo) over cz
        fine_line(oz, c, r);
        // only the rows and planes that are read are written (whole x rows: 64-byte pieces)
#pragma unroll
        for (int m = 0; m < 8; ++m)
            if (row_needed && ((need >> (8 + m)) & 1)) put_virtual<NT>(&out[v * out_stride + m * (NPT * NPT)], r[m]);
        __builtin_amdgcn_wave_barrier();                         // the next variable's x pass overwrites the array
    }
}

// Virtual blocks with the centred ghost rule.  The value at a fine position inside a leaf L that is one level coarser
// is the centred six-point stencil on the coarse lattice around it, nodes c0 - 2 .. c0 + 3 with c0 = f / 2, and nodes
// outside L are ghost points of L.  A child octant o of L therefore needs, per axis, the nine coarse nodes
// 4 o - 2 .. 4 o + 6: a 9^3 part of L's padded block, which is gathered here straight from the zipped array (729
// sources).  None of them lies in another virtual block, so one launch fills them all: a virtual block is needed because
// some block touches the octant, that block's parent P is a same-level neighbour of L, and the seven neighbours of L on
// the octant's side are 26-neighbours of P too (per axis they step back towards P where L is off P, and one to either
// side where it is not); P is subdivided, so the 2:1 balance leaves none of them coarser than L.
// Then the same three passes as in k_virtual, with nine nodes per line; a wavefront owns one variable of one virtual block at
// a time and requests its nodes in the order of the storage, a few lines per load, through its staging array (a lane that gathers whole
// x lines touches 64 lines of the cache per load, which bound that form: the L1 takes one per cycle).  What differs is who works out
// the 729 sources:
//   k_virtual_centred       nine variables or more: the eight wavefronts of a workgroup share one virtual block, and its sources.
//   k_virtual_centred_few   up to eight: each wavefront by itself, from a table made at compile time and L's row of the ghost table, so
//       that a workgroup can take several virtual blocks and nothing needs a workgroup barrier.
// (us, unzip_centred on 21,064 blocks, of which the fill of 11,056 virtual blocks, with the sources worked out together / by each wavefront:
// 5 variables 898 / 877, 6: 1075 / 1056, 8: 1425 / 1405; up to four, with gathered lines / as here: 1: 136 / 134, 2: 279 / 268, 4: 711 / 688.
// Steps of the wave system 1652 -> 1585 on 47,783 blocks, 60.7 -> 56.5 on 834; of Burgers 789 -> 750, 44.0 -> 40.1.)
constexpr int CN = 9;                                // coarse nodes per axis

// the eight fine values of a line with nine nodes v (node n is coarse node 4 o - 2 + n): even f passes node c0 through,
// odd f takes nodes c0 - 2 .. c0 + 3 with the centred weights, acc = w0 v, then five fma (as centred_line)
__device__ __forceinline__ void fine_line_centred(const double (&v)[CN], double (&r)[8])
{
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        r[2 * n] = v[n + 2];
        double acc = c_lag[12] * v[n];
#pragma unroll
        for (int m = 1; m < 6; ++m) acc = fma(c_lag[12 + m], v[n + m], acc);
        r[2 * n + 1] = acc;
    }
}

constexpr int CRS = CN, CPS = CN * CN + 7;           // row and plane stride of the staging array of nodes: 88 = 24 (mod 32)
// x pass over a wavefront's staging array of nodes: lines (cz, cy), 81 of them; in place (a lane writes the first eight positions of the
// row it has read)
__device__ __forceinline__ void centred_x(double* A, int lane)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int line = lane + 64 * h;
        if (line < CN * CN) {
            double* row = A + line * CRS + 7 * (line / CN);
            double c[CN], r[8];
#pragma unroll
            for (int m = 0; m < CN; ++m) c[m] = row[m];
            fine_line_centred(c, r);
#pragma unroll
            for (int m = 0; m < 8; ++m) row[m] = r[m];
        }
    }
}

// y and z passes of a wavefront's staging array A, in which the x pass has left lines of eight fine values, rows RSTR and
// planes PSTR apart; writes the rows and planes in `need` to the virtual block at `out` (the lane's value of its plane 0)
template <int RSTR, int PSTR, bool NT>
__device__ __forceinline__ void centred_yz(double* A, double* out, int need, int lane)
{
    double c[CN], r[8];
    // y pass: lines (cz, tx), 72 of them; in place
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int line = lane + 64 * h;
        if (line < CN * 8) {
            double* col = A + (line >> 3) * PSTR + (line & 7);
#pragma unroll
            for (int m = 0; m < CN; ++m) c[m] = col[m * RSTR];
            fine_line_centred(c, r);
#pragma unroll
            for (int m = 0; m < 8; ++m) col[m * RSTR] = r[m];
        }
    }
    __builtin_amdgcn_wave_barrier();
    // z pass: lines (ty, tx) = (hi, lo)
    const int hi = lane >> 3, lo = lane & 7;
#pragma unroll
    for (int m = 0; m < CN; ++m) c[m] = A[m * PSTR + hi * RSTR + lo];
    fine_line_centred(c, r);
#pragma unroll
    for (int m = 0; m < 8; ++m)
        if (((need >> hi) & 1) && ((need >> (8 + m)) & 1)) put_virtual<NT>(&out[m * (NPT * NPT)], r[m]);
    __builtin_amdgcn_wave_barrier();                 // the next variable overwrites the array
}

constexpr int kFewVariables = 8;                     // up to here k_virtual_centred_few
template <bool NT>
__global__ __launch_bounds__(NTHREADS) void k_virtual_centred(DeviceTree tr, int nvar, const double* __restrict__ zipped,
                                                              double* __restrict__ virt)
{
    __shared__ double staging[8][CN * CPS];
    __shared__ uint32_t plan[CN * CN * CN];          // byte offsets of the 729 sources
    __shared__ int32_t gt[27 * 5];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int64_t q = block_of_workgroup(blockIdx.x), nb = tr.nb;
    if (q >= tr.n_virt) return;                      // uniform over the workgroup
    const int64_t leaf = tr.vblk[2 * q];
    const int oct = tr.vblk[2 * q + 1];
    const int need = tr.vneed[q];                    // y rows and z planes that any block reads
    if (tid < 27 * 5) gt[tid] = tr.ghost_v[leaf * (27 * 5) + tid];
    __syncthreads();
    for (int p = tid; p < CN * CN * CN; p += NTHREADS) {
        const int nz = p / (CN * CN), r = p - nz * CN * CN, ny = r / CN, nx = r - ny * CN;
        // position in L's padded block: coarse node 4 o - 2 + n, shifted by the three ghost layers
        const int ii = 4 * (oct & 1) + 1 + nx, jj = 4 * ((oct >> 1) & 1) + 1 + ny, kk = 4 * (oct >> 2) + 1 + nz;
        const int rx = ii < PAD ? 0 : (ii < PAD + NPT ? 1 : 2);
        const int ry = jj < PAD ? 0 : (jj < PAD + NPT ? 1 : 2);
        const int rz = kk < PAD ? 0 : (kk < PAD + NPT ? 1 : 2);
        const int lx = ii - PAD + (1 - rx) * NPT, ly = jj - PAD + (1 - ry) * NPT, lz = kk - PAD + (1 - rz) * NPT;
        plan[p] = ghost_source(&gt[(rz * 9 + ry * 3 + rx) * 5], rx, ry, rz, lx, ly, lz);   // the centre entry is L itself
    }
    __syncthreads();
    double* A = staging[wave];
    const int64_t in_stride = nb * BLK, out_stride = tr.n_virt * BLK;
    double* out = virt + q * BLK + lane;
    // this lane's share of the gather: elements lane, lane + 64, ... of the 729 (the lanes past it repeat the last one)
    constexpr int NG = (CN * CN * CN + 63) / 64;     // 12
    uint32_t off[NG];
    int dst[NG];
#pragma unroll
    for (int m = 0; m < NG; ++m) {
        const int p = min(lane + 64 * m, CN * CN * CN - 1);
        off[m] = plan[p];
        dst[m] = p + 7 * (p / (CN * CN));
    }
    double nxt[NG];
    auto gather = [&](int v) {
        const double* base = zipped + v * in_stride;
#pragma unroll
        for (int m = 0; m < NG; ++m) nxt[m] = ldg(base, off[m]);
    };
    if (wave < nvar) gather(wave);
#pragma unroll 1
    for (int v = wave; v < nvar; v += 8) {
#pragma unroll
        for (int m = 0; m < NG; ++m) A[dst[m]] = nxt[m];
        if (v + 8 < nvar) gather(v + 8);
        __builtin_amdgcn_wave_barrier();
        centred_x(A, lane);
        __builtin_amdgcn_wave_barrier();
        centred_yz<CRS, CPS, NT>(A, out + v * out_stride, need, lane);
    }
}

// Virtual blocks per workgroup of k_virtual_centred_few: as its wavefronts have variables for, halved as long as the 256
// compute units can hold all workgroups at once, three each by their LDS (us, step with the centred rule, always 8 or 4 / as here / with half
// as many workgroups / with twice as many: Burgers 39.2 / 33.2 / 33.6 / 33.8 on 554 blocks, 42.2 / 37.6 / 37.1 / 37.5 on 708, 48.0 / 46.0 /
// 47.0 / 52.1 on 1,170; wave system 48.4 / 42.8 / 42.9 / 42.9, 53.2 / 50.2 / 49.2 / 50.5, 73.2 / 69.4 / 73.2 / 75.0).
inline int centred_per_workgroup(int64_t n_virt, int nvar)
{
    int per = 8 / nvar;
    while (per > 1 && n_virt <= 3 * 256 * (int64_t)(per / 2)) per /= 2;
    return per;
}
// Sources of the 729 nodes for each child octant of L, worked out at compile time but for the table row of L: which of the eight
// directions on the octant's side (bit per axis on which the node is beyond L), which finer neighbour there, the node's index in a
// neighbour of the same level and in a finer one.
constexpr int CNODES = CN * CN * CN, CITEMS = (CNODES + 63) / 64;              // 729; 12 per lane
struct CentredItems { uint32_t at[8][CITEMS * 64]; };
constexpr CentredItems make_centred_items()
{
    CentredItems t{};
    for (int oct = 0; oct < 8; ++oct)
        for (int n = 0; n < CITEMS * 64; ++n) {
            const int p = n < CNODES ? n : CNODES - 1;                         // the lanes past them repeat the last one
            const int node[3] = {p % CN, p / CN % CN, p / (CN * CN)};
            int out = 0, q = 0, sh = 0, same = 0, fine = 0;
            for (int a = 0; a < 3; ++a) {
                const int f = 4 * ((oct >> a) & 1) - 2 + node[a];              // in L: 0..7
                const int l = f < 0 ? f + NPT : (f < NPT ? f : f - NPT);       // in the octant of L's size that holds it
                const int half = f < 0 ? 1 : (f < NPT ? l >> 2 : 0);           // the half of it in which a finer neighbour holds it
                if (f < 0 || f >= NPT) out |= 1 << a;
                else { q |= half << sh; ++sh; }
                same |= l << (3 * a);
                fine |= (2 * l - NPT * half) << (3 * a);
            }
            if (out == 0) q = 0;                                               // L itself
            t.at[oct][n] = (uint32_t)(out * 4 + q) | (uint32_t)same << 5 | (uint32_t)fine << 14;
        }
    return t;
}
__device__ const CentredItems kCentredItems = make_centred_items();

template <bool NT>
__global__ __launch_bounds__(NTHREADS) void k_virtual_centred_few(DeviceTree tr, int nvar, int per, const double* __restrict__ zipped,
                                                                  double* __restrict__ virt)
{
    __shared__ double staging[8][CN * CPS];
    __shared__ uint32_t rows[8][8 * 4];              // L's neighbours in the eight directions, four each (kFinerLeaf: of which the node needs one)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int sub = wave / nvar, v = wave - sub * nvar;         // which of the workgroup's `per` virtual blocks, variable
    const int64_t q = block_of_workgroup(blockIdx.x) * per + sub, nb = tr.nb;
    if (sub >= per || q >= tr.n_virt) return;        // uniform over the wavefront; the kernel has no workgroup barrier
    const int64_t leaf = tr.vblk[2 * q];
    const int oct = tr.vblk[2 * q + 1];
    const int need = tr.vneed[q];                    // y rows and z planes that any block reads
    uint32_t item[CITEMS];
#pragma unroll
    for (int m = 0; m < CITEMS; ++m) item[m] = kCentredItems.at[oct][lane + 64 * m];
    uint32_t* row = rows[wave];
    constexpr uint32_t kFinerLeaf = 1u << 31;
    if (lane < 8 * 4) {
        const int out = lane >> 2;
        const int dx = out & 1 ? 2 * (oct & 1) - 1 : 0, dy = out & 2 ? (oct & 2) - 1 : 0, dz = out & 4 ? (oct >> 1 & 2) - 1 : 0;
        const int32_t* e = &tr.ghost_v[leaf * (27 * 5) + (13 + 9 * dz + 3 * dy + dx) * 5];               // the centre entry is L itself
        const int32_t kind = e[0], first = e[1], own = e[1 + (lane & 3)];
        row[lane] = kind == K_SAME ? (uint32_t)first : (uint32_t)own | kFinerLeaf;
    }
    __builtin_amdgcn_wave_barrier();
    const double* base = zipped + v * nb * BLK;
    uint32_t id[CITEMS];
    double node[CITEMS];
#pragma unroll
    for (int m = 0; m < CITEMS; ++m) id[m] = row[item[m] & 31];
#pragma unroll
    for (int m = 0; m < CITEMS; ++m) node[m] = ldg(base, (id[m] * BLK + (id[m] & kFinerLeaf ? item[m] >> 14 : item[m] >> 5) % BLK) * 8u);
    double* A = staging[wave];
#pragma unroll
    for (int m = 0; m < CITEMS; ++m) {
        const int p = min(lane + 64 * m, CNODES - 1);
        A[p + 7 * (p / (CN * CN))] = node[m];
    }
    __builtin_amdgcn_wave_barrier();
    centred_x(A, lane);
    centred_yz<CRS, CPS, NT>(A, virt + v * tr.n_virt * BLK + q * BLK + lane, need, lane);
}

template <bool STREAM>
__global__ __launch_bounds__(NTHREADS) void k_zip(int64_t nblocks, const double* __restrict__ padded, double* __restrict__ zipped)
{
    const int tid = threadIdx.x;
    const int64_t q = blockIdx.x;   // var*nb + block
    if (q >= nblocks) return;
    const int i = tid & 7, j = (tid >> 3) & 7, k = tid >> 6;
    zipped[q * BLK + tid] = padded[q * PBLK + ((k + PAD) * NP + (j + PAD)) * NP + (i + PAD)];
}

// The same in 16-byte words and past the caches, from kStreamZipBlocks on.  What bounds it is memory: of the lines that hold a padded block's
// interior 43 % are ghosts.  (us a call on changing buffers, plain / non-temporal, then with a reduction over the result behind each, and the pipeline
// of unzip, rhs_eval and this: DERIVS on 1,919 blocks, 7,676 of a variable, 16.9 / 15.8, 31.6 / 32.2, 68.4 / 60.5; wave 6,792: 14.3 / 13.9, 28.7 /
// 29.9, 122 / 114, 10,460: 24.5 / 21.0, 39.1 / 39.3, 185 / 170; on 47,783 blocks wave 203 / 180, 277 / 252, 1607 / 1564, DERIVS 408 / 365, 550 / 504,
// 1666 / 1573; 24 variables on 512 blocks 28.8 / 24.3, 43.5 / 43.7, 198 / 191, on 21,064 1075 / 972, 1423 / 1321, 8602 / 8508.  With 8-byte
// words 2 to 8 % slower up to 9,213 blocks and the same beyond; 16-byte words without the rest 1 to 3 % slower on large trees.)
constexpr int64_t kStreamZipBlocks = 8192;           // of all variables
template <>
__global__ __launch_bounds__(BLK / 2) void k_zip<true>(int64_t nblocks, const double* __restrict__ padded, double* __restrict__ zipped)
{
    const int tid = threadIdx.x;
    const int64_t q = blockIdx.x;   // var*nb + block
    if (q >= nblocks) return;
    const int i = 2 * (tid & 3), j = (tid >> 2) & 7, k = tid >> 5;
    const Pair v = __builtin_nontemporal_load(reinterpret_cast<const PairAt8*>(padded + q * PBLK + ((k + PAD) * NP + (j + PAD)) * NP + (i + PAD)));
    __builtin_nontemporal_store(v, reinterpret_cast<PairAt8*>(zipped + q * BLK + 2 * tid));
}

// Non-temporal accesses cost where what a launch writes would have been in the memory-side cache for the next one: in a step,
// whose stages read each other's vectors, below about the size of that cache; after an evaluation, if its result is read
// next.  They pay everywhere else, and for the launch itself at every size.  Measured, us without / with (kernels.hpp has the
// sizes at which both are the same): steps of the wave system 231 / 252 on 6,791 blocks (223 MB), 306 / 304 on 8,716 (286 MB),
// 381 / 362 on 10,550 (346 MB), 1645 / 1501 on 47,783; steps of Burgers 253 / 256 on 15,324 blocks (251 MB), 351 / 332 on 21,120
// (346 MB); evaluations on new buffers, then alone / with a pass over the result: DERIVS 46.1 / 35.1 on 7,141 blocks (146 MB),
// 79.6 / 77.0 on 7,813; wave 65.6 / 63.2 and 104.8 / 102.1 on 9,780 (160 MB); Burgers 59.8 / 55.8 and 96.6 / 93.4 on 19,580 (160 MB).
template <int KIND, int EPI>
bool streams(int64_t nb)
{
    const int64_t vector = nb * BLK * (int64_t)sizeof(double);
    const ot_rhs_kind kind = static_cast<ot_rhs_kind>(KIND);
    return EPI == kOutZipped ? (ot_rhs_nvar_in(kind) + ot_rhs_nvar_out(kind)) * vector > kStreamEvalBytes
                             : 4 * ot_rhs_nvar_in(kind) * vector > kStreamStepBytes;
}

// On padded blocks only the result's 64 bytes of every 112 are written, which the L2 and the memory-side cache complete from memory
// unless the line is there.  Non-temporal stores are worth it from where input and output leave that cache (us a call on changing
// buffers, plain / non-temporal, and the pipeline of unzip, this and zip: Burgers on 1,919 blocks, 84 MB, 9.6 / 10.2, 34.6 / 34.8, on 3,396, 149
// MB, 16.7 / 15.5, 62.7 / 63.8, on 5,230, 230 MB, 35.6 / 25.5, 95.4 / 92.6; wave 168 MB 19.6 / 17.9, 71.4 / 71.9, 298 MB 48.9 / 39.3, 122.5 /
// 118.1, on 47,783 698 / 576, 1613 / 1498; DERIVS 211 MB 19.9 / 27.3, 68.5 / 72.2, 373 MB 63.0 / 45.1, 123.7 / 117.8, on 47,783 879 / 720,
// 1662 / 1511).
constexpr int64_t kStreamPaddedBytes = 256ll << 20;

template <int KIND, bool ZIN, int EPI>
hipError_t launch_one(const DeviceTree& t, const RhsArgs& a, hipStream_t s)
{
    if constexpr (KIND == OT_RHS_SYN24) {
        // bricks reach 2^20 virtual blocks, whatever the alignment of the arrays (us, a thread per point / bricks, evaluation and step on 792 blocks
        // 108 / 93, 512 / 457, on 21,057 2141 / 1838, 10,780 / 9332; arrays aligned to 8 bytes only 107 / 94, 523 / 461, 2178 / 1867, 10,907 / 9434)
        return ZIN && t.n_virt > kBlockLimit ? launch_rhs_pairs(t, static_cast<Epilogue>(EPI), a, s) : launch_rhs_bricks(t, static_cast<Epilogue>(EPI), a, s);
    } else {
        if constexpr (ZIN) {
            if (streams<KIND, EPI>(t.nb)) {
                hipLaunchKernelGGL((k_rhs_stream<KIND, EPI>), dim3(grid_for_blocks<kStreamChunk>(t.nb)), dim3(rhs_threads(KIND)), 0, s, t, a);
                return hipGetLastError();
            }
        }
        if constexpr (!ZIN) {
            constexpr ot_rhs_kind kind = static_cast<ot_rhs_kind>(KIND);
            if ((ot_rhs_nvar_in(kind) + ot_rhs_nvar_out(kind)) * t.nb * PBLK * (int64_t)sizeof(double) > kStreamPaddedBytes) {
                hipLaunchKernelGGL((k_rhs_padded_stream<KIND>), dim3(grid_for_blocks(t.nb)), dim3(rhs_threads(KIND)), 0, s, t, a);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((k_rhs<KIND, ZIN, EPI>), dim3(grid_for_blocks(t.nb)), dim3(rhs_threads(KIND)), 0, s, t, a);
        return hipGetLastError();
    }
}

template <int KIND>
hipError_t launch_kind(const DeviceTree& t, bool zin, Epilogue ep, const RhsArgs& a, hipStream_t s)
{
    if (zin && !a.virt && t.n_virt > 0) return hipErrorInvalidValue;
    if (zin && ep == kRkFirst && a.in != a.u) return hipErrorInvalidValue;   // the first stage takes the state from its input tiles
    if (!zin) {
        if (ep != kOutPadded) return hipErrorInvalidValue;
        return launch_one<KIND, false, kOutPadded>(t, a, s);
    }
    if constexpr (KIND != OT_RHS_DERIVS) {           // its output is not a rate of change of its input: no stages
        switch (ep) {
        case kRkFirst: return launch_one<KIND, true, kRkFirst>(t, a, s);
        case kRkMiddle: return launch_one<KIND, true, kRkMiddle>(t, a, s);
        case kRkLast: return launch_one<KIND, true, kRkLast>(t, a, s);
        default: break;
        }
    }
    return ep == kOutZipped ? launch_one<KIND, true, kOutZipped>(t, a, s) : hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_unzip(const DeviceTree& t, int nvar, const double* zipped, const double* virt, double* padded, hipStream_t s)
{
    if (t.nb <= 0 || nvar <= 0) return hipSuccess;
    if (!virt && t.n_virt > 0) return hipErrorInvalidValue;
    const int stride = unzip_stride(t.nb, nvar);
    hipLaunchKernelGGL(k_unzip, dim3(grid_for_blocks(t.nb), (unsigned)stride), dim3(NTHREADS), 0, s, t, nvar, stride, zipped, virt, padded);
    return hipGetLastError();
}

hipError_t launch_virtual(const DeviceTree& t, int nvar, const double* zipped, double* virt, hipStream_t s)
{
    if (t.n_virt <= 0 || nvar <= 0) return hipSuccess;
    const int per = 8 / (nvar < 8 ? nvar : 8);       // virtual blocks per workgroup, as in the kernel
    hipLaunchKernelGGL(fill_streams(t, nvar) ? k_virtual<true> : k_virtual<false>, dim3(grid_for_blocks((t.n_virt + per - 1) / per)), dim3(NTHREADS), 0, s, t, nvar, zipped, virt);
    return hipGetLastError();
}

hipError_t launch_virtual_centred(const DeviceTree& t, int nvar, const double* zipped, double* virt, hipStream_t s)
{
    if (t.n_virt <= 0 || nvar <= 0) return hipSuccess;
    if (nvar > kFewVariables) {
        hipLaunchKernelGGL(fill_streams(t, nvar) ? k_virtual_centred<true> : k_virtual_centred<false>, dim3(grid_for_blocks(t.n_virt)), dim3(NTHREADS), 0, s, t, nvar, zipped, virt);
    } else {
        const int per = centred_per_workgroup(t.n_virt, nvar);
        hipLaunchKernelGGL(fill_streams(t, nvar) ? k_virtual_centred_few<true> : k_virtual_centred_few<false>, dim3(grid_for_blocks((t.n_virt + per - 1) / per)), dim3(NTHREADS), 0, s, t, nvar, per, zipped, virt);
    }
    return hipGetLastError();
}

hipError_t launch_zip(const DeviceTree& t, int nvar, const double* padded, double* zipped, hipStream_t s)
{
    const int64_t n = t.nb * nvar;
    if (n <= 0) return hipSuccess;
    if (n >= kStreamZipBlocks) hipLaunchKernelGGL(k_zip<true>, dim3((unsigned)n), dim3(BLK / 2), 0, s, n, padded, zipped);
    else hipLaunchKernelGGL(k_zip<false>, dim3((unsigned)n), dim3(NTHREADS), 0, s, n, padded, zipped);
    return hipGetLastError();
}

hipError_t launch_rhs(const DeviceTree& t, ot_rhs_kind kind, bool in_zipped, Epilogue ep, const RhsArgs& args, hipStream_t s)
{
    if (t.nb <= 0) return hipSuccess;
    switch (kind) {
    case OT_RHS_DERIVS: return launch_kind<OT_RHS_DERIVS>(t, in_zipped, ep, args, s);
    case OT_RHS_WAVE: return launch_kind<OT_RHS_WAVE>(t, in_zipped, ep, args, s);
    case OT_RHS_BURGERS: return launch_kind<OT_RHS_BURGERS>(t, in_zipped, ep, args, s);
    case OT_RHS_SYN24: return launch_kind<OT_RHS_SYN24>(t, in_zipped, ep, args, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace octfd
