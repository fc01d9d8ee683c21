// Launch interface between the C ABI (capi.cpp) and the gfx950 kernels (kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "octfd.h"
#include "table_rows.hpp"

namespace octfd {

struct DeviceTree {
    const ot_leaf* leaves;   // [nb]
    int64_t nb;
    // virtual blocks (see HostTree): the ghost table that names them and what each is
    const int32_t* ghost_v;  // [nb][27][5]
    const int32_t* vblk;     // [n_virt][2] {source leaf, child octant} of every virtual block
    int64_t n_virt;
    // the 24-field system on zipped input: the work units of the two-block kernel (see HostTree::units)
    const int32_t* units;
    int64_t n_units;
    const int32_t* vneed;    // [n_virt] y rows (bits 0..7) and z planes (bits 8..15) of a virtual block that are read at all
};

constexpr int32_t kUnitSingle = 1 << 30;   // flag on a unit: one block without a partner

// From which size of a step's four vectors (an evaluation's input and output) kernels write, and where that pays read,
// non-temporally.  Sizes at which the two ways take the same time, measured on trees around two centres (MB; virtual blocks,
// which share the 256 MB memory-side cache, not counted):
//   steps                     wave 286, Burgers 220 to 265, 24 fields 305 to 330 (brick.hip)
//   with the centred rule     wave 312, Burgers 259, 24 fields 340 to 390
//   evaluations by themselves: below 100, 24 fields below 130 (non-temporal / plain there 0.78 to 0.99, at 290 MB 0.77 to 0.96)
//   evaluations, the result read by the next launch: DERIVS 115 to 160, wave 75 to 90, Burgers below 60, 24 fields up to 145
// The line for steps lies in the middle of these: on its wrong side a step loses at most 4 % (Burgers, 301 MB) and 2 % (24
// fields with the centred rule, 327 MB).  The line for evaluations lies at the top of the last range.  New buffers each call,
// plain / non-temporal, us, by themselves and with a reduction over the result behind each:
//   DERIVS     59 MB 20.4 / 17.3, 31.1 / 31.1    144 MB 47.5 / 34.0, 64.5 / 66.9    158 MB 51.0 / 36.5, 69.4 / 71.6    189 MB 58.4 / 42.5, 79.6 / 82.0
//   wave      151 MB 64.6 / 60.1, 74.6 / 76.2    177 MB 74.2 / 69.6, 85.3 / 87.4    Burgers 139 MB 55.0 / 50.5, 65.5 / 66.0
//   24 fields 110 MB 82.6 / 79.4, 93.3 / 95.7    154 MB 95.1 / 90.9, 106.5 / 108.0    171 MB 98.7 / 95.8, 113.6 / 114.5
// so above it a caller who reduces the result at once pays up to 3 %, and any other gains 3 to 28 %.  Another run of the same, on four sets of buffers in
// turn, saw nothing of those 3 %: DERIVS 162 MB 49.6 / 38.2, 76.4 / 75.5, 175 MB 53.0 / 41.1, 80.9 / 80.5, 187 MB 55.9 / 42.8, 85.2 / 83.9; wave
// 162 MB 63.4 / 61.2, 83.2 / 84.1, 187 MB 71.5 / 67.5, 92.9 / 92.4; Burgers 161 MB 58.1 / 54.0, 77.7 / 76.7; 24 fields 162 MB 97.2 / 94.7, 117.2 / 118.4.
constexpr int64_t kStreamStepBytes = 300ll << 20, kStreamEvalBytes = 160000000;

// workgroup i runs on XCD i mod kXcds; the kernels deal chunks of kChunk consecutive blocks to the XCDs in turn
constexpr int kSchedChunk = 16;
constexpr int kSchedXcds = 8;

// how the right-hand side leaves the kernel
enum Epilogue : int {
    kOutPadded = 0,   // interior of a padded-shaped array
    kOutZipped = 1,   // zipped array
    kRkFirst = 2,     // acc = k;        stage = fma(c, k, u)        (u is the kernel's input)
    kRkMiddle = 3,    // acc = acc + 2k; stage = fma(c, k, u)
    kRkLast = 4       // u = fma(c, acc + k, u)
};

struct RhsArgs {
    const double* in;   // padded [V][nb][2744] or zipped [V][nb][512]
    double* out;        // kOutPadded / kOutZipped: result; kRkFirst / kRkMiddle: next stage vector
    double* acc;        // Runge-Kutta accumulator (zipped)
    double* u;          // state at the start of the step (zipped); written by kRkLast
    const double* virt;      // zipped input: the virtual blocks of `in`, [V][n_virt][512], filled by launch_virtual or
                             // launch_virtual_centred (which of the two decides the ghost rule)
    double c;           // dt/2, dt or dt/6
    double sigma;       // Kreiss-Oliger strength
};

// the ghost table of nb blocks on the device, coarser neighbours as virtual blocks
hipError_t launch_ghost_table(const TableSource& t, int64_t nb, int32_t* ghost_v, hipStream_t s);
// padded [nvar][nb][2744] from zipped and its virtual blocks (filled by one of the two calls below: which one decides
// the ghost rule)
hipError_t launch_unzip(const DeviceTree& t, int nvar, const double* zipped, const double* virt, double* padded, hipStream_t s);
// fills the virtual blocks of a zipped array: virt [nvar][n_virt][512], each the child octant of its source leaf,
// every point interpolated inside that leaf exactly as a ghost point is in unzip ...
hipError_t launch_virtual(const DeviceTree& t, int nvar, const double* zipped, double* virt, hipStream_t s);
// ... or in unzip_centred
hipError_t launch_virtual_centred(const DeviceTree& t, int nvar, const double* zipped, double* virt, hipStream_t s);
hipError_t launch_zip(const DeviceTree& t, int nvar, const double* padded, double* zipped, hipStream_t s);
// the 24-field right-hand side over the units of the tree, two points per thread (brick.hip): zipped input of trees with at most 2^20 virtual
// blocks, epilogue kOutZipped or one of the Runge-Kutta stages, or padded input of any tree, epilogue kOutPadded
hipError_t launch_rhs_bricks(const DeviceTree& t, Epilogue ep, const RhsArgs& args, hipStream_t s);
// a thread per point (pair.hip): zipped input of any tree
hipError_t launch_rhs_pairs(const DeviceTree& t, Epilogue ep, const RhsArgs& args, hipStream_t s);
// in_zipped = false: args.in is padded; true: args.in is zipped and args.virt holds its virtual blocks
hipError_t launch_rhs(const DeviceTree& t, ot_rhs_kind kind, bool in_zipped, Epilogue ep, const RhsArgs& args, hipStream_t s);

}  // namespace octfd
