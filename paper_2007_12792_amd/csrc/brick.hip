// gfx950 kernel of the 24-field right-hand side, on zipped or padded input: two sibling blocks (a 16 x 8 x 8 brick, see pair.hip) per
// workgroup of 512 threads, TWO x neighbours per thread, one workgroup at a time on every compute unit (rounds.hpp).
//
// What bounded the kernel with a thread per point: LDS reads of 8 bytes (42 % of the time), vector instructions (36 %), and that the
// two hardly overlap, all wavefronts of the compute unit being in the same phase of a pass.  Two points per thread halve the first:
// the compute unit reads 16-byte words from LDS at 230 to 250 bytes per cycle where 8-byte words come at 128, and a pair
// shares its x taps.  256 registers a thread take what memory and LDS were read for before, and data requested further ahead:
//   - second derivatives in LDS (Lap, 80 KB); all ten pointwise fields and what u_{a+11} needs of the later passes in registers, so
//     that u_{a+11} is read again in ten passes of 24 only;
//   - in the passes without second derivatives, two tiles in turn (the second where D1_y u, D1_z u lie otherwise), one barrier, and
//     the data of the variable after the next one on its way: such a pass is shorter than the way to memory;
//   - a workgroup goes from unit to unit through its part of the launch, and the first data of the next is requested in the last passes of the
//     one before;
//   - loads are spread over a pass: issued at once they wait for each other at the L1 (64 bytes per cycle).
// Every ghost item is a pair too (a 16-byte load where its neighbour is of the same level, two where it is finer), its place and
// source worked out at compile time but for the table row.  Powers of two are moved out of the arithmetic where that changes
// no rounding (short of underflow, and of overflow: within a factor of eight of it in products of fields, and where sigma itself, times up to
// 2^16, passes it): 104 instead of 116 fp64 instructions in a pass without, 200 instead of 240 in one with second derivatives.
// (us, thread per point -> here: step on 102,075 blocks 50,750 -> 43,500, on 21,064 10,920 -> 9,510, on 792 503 -> 442, on 526 399 -> 353;
// evaluation on 21,064 blocks 2170 -> 1880, on 526 94 -> 82.  Of these: pairs and 16-byte words alone 10,150 for the step on 21,064
// blocks, powers of two and compile-time items 10,120, pairs throughout and two passes ahead 9,680, from unit to unit 9,640, loads spread
// 9,510.  With three chains of gradients instead of Lap in LDS, u_{a+11} never read again and one barrier per pass 10,750: 27 passes
// instead of 25, and no registers left to request data two passes ahead.)
#include "kernels.hpp"
#include "rounds.hpp"
#include "stencils.hpp"
#include "syn24.hpp"
#include "tile.hpp"

#include <type_traits>

namespace octfd {
namespace {

namespace br {
constexpr int NT = 512;
constexpr int RS = 24;                   // row stride, 8 * odd: four rows of four pairs fall into different 16-byte banks
constexpr int PS = NP * RS + 2;          // plane stride 338: so do columns of points (j, k) (ns per 16-byte read of a wavefront, own points /
                                         // columns / rows of planes: 2.4 / 2.4 / 3.6; stride 336 2.7 / 6.8 / 2.4, 340 2.1 / 3.6 / 5.1)
constexpr int X0 = 1;                    // position of tile column 0 in its row: own pairs start at even positions
constexpr int TILE = NP * PS;            // 4732
constexpr int WZ = NPT * PS;             // D1_z u on [8 k][14 jj][22 ii]
constexpr int YPS = NPT * RS + 18;       // 210
constexpr int WY = NPT * YPS;            // D1_y u on [8 k][8 j][22 ii]
constexpr int BUF = TILE > WZ + WY ? TILE : WZ + WY;   // the D1 arrays, or the second tile

constexpr bool gz_inside(int g) { return g >= PAD && g < PAD + NPT; }
constexpr int gyz(int g) { return g < PAD ? g : g + NPT; }        // 0,1,2,11,12,13
constexpr int at(int kk, int jj, int ii) { return kk * PS + jj * RS + ii + X0; }

// A task is 64 lanes' worth of ghost items, each a pair of x neighbours.  Task 8 m + w is item m of wavefront w.
//   0..5 y faces, 6..11 z faces, 12..15 x faces, 16..26 yz, xy and xz edges (the last task half)
// Of the three ghost columns beyond an x face the pair next to the brick and one further are taken, whose outermost value lands in
// the padding of the row.
constexpr int FACE_ITEMS = 2, ITEMS = 4, LAST_ITEM_WAVES = 3, EDGE_PAIRS = 288 + 192 + 192;
struct Point3 { int ii, jj, kk; };
constexpr int gx_pair(int c) { return 2 * (c & 1) - 1 + (c & 2 ? 2 * NPT + PAD + 1 : 0); }     // -1, 1, 19, 21
constexpr Point3 ghost_item(int task, int lane)
{
    if (task < 6) {
        const int q = task * 64 + lane, r = q >> 3, kq = r / 6;
        return {PAD + 2 * (q & 7), gyz(r - 6 * kq), PAD + kq};
    }
    if (task < 12) return {PAD + 2 * (lane & 7), PAD + (lane >> 3), gyz(task - 6)};
    if (task < 16) {
        const int q = (task - 12) * 64 + lane, r = q >> 2;
        return {gx_pair(q & 3), PAD + (r & 7), PAD + (r >> 3)};
    }
    int q = (task - 16) * 64 + lane < EDGE_PAIRS ? (task - 16) * 64 + lane : EDGE_PAIRS - 1;
    if (q < 288) {
        const int r = q >> 3, kg = r / 6;
        return {PAD + 2 * (q & 7), gyz(r - 6 * kg), gyz(kg)};
    }
    q -= 288;
    if (q < 192) {
        const int r = q >> 2, kq = r / 6;
        return {gx_pair(q & 3), gyz(r - 6 * kq), PAD + kq};
    }
    const int r = (q - 192) >> 2;
    return {gx_pair(q & 3), PAD + (r & 7), gyz(r >> 3)};
}

// An item, worked out at compile time: which entry of the two blocks' table rows says where it comes from, which of up to four finer
// neighbours holds it, the (first) value's index in a block of the same level and in a finer one, and where it goes in the tile.
// kFixed: it has no meaning (behind the ghost columns of a block without a partner) and takes the block's first values.
struct Item { uint32_t where, dst; };
constexpr uint32_t kFixed = 1u << 31;
// On padded input: the index of the pair's first value in the unit's two padded blocks, which follow each other; without a meaning, that of
// the block's first own value.
constexpr uint32_t padded_index(int kk, int jj, int ii) { return (uint32_t)((kk * NP + jj) * NP + ii); }
constexpr uint32_t padded_source(bool single, Point3 p)
{
    const bool upper = p.ii >= PAD + NPT;
    if (!(single && upper)) return (upper ? PBLK : 0) + padded_index(p.kk, p.jj, p.ii - (upper ? NPT : 0));
    // the upper half of a block without a partner: its ghosts beyond the x face, as far as stencils along the axes and xz, xy edges read them
    const bool meant = p.ii < 2 * PAD + NPT && (gz_inside(p.kk) || gz_inside(p.jj));
    return meant ? padded_index(p.kk, p.jj, p.ii) : padded_index(PAD, PAD, PAD);
}
constexpr Item make_item(bool single, int task, int lane)
{
    const Point3 p = ghost_item(task, lane);
    int h = p.ii >= PAD + NPT ? 1 : 0;
    int rx = h ? (p.ii < PAD + 2 * NPT ? 1 : 2) : (p.ii < PAD ? 0 : 1);
    const int ry = p.jj < PAD ? 0 : (p.jj < PAD + NPT ? 1 : 2), rz = p.kk < PAD ? 0 : (p.kk < PAD + NPT ? 1 : 2);
    int lx = p.ii - PAD - NPT * h + (1 - rx) * NPT;
    const int ly = p.jj - PAD + (1 - ry) * NPT, lz = p.kk - PAD + (1 - rz) * NPT;
    const uint32_t dst = (uint32_t)at(p.kk, p.jj, p.ii);
    if (single && h) {
        if (p.ii >= 2 * PAD + NPT) return {kFixed, dst};
        h = 0; rx = 2; lx = p.ii - PAD - NPT;
    }
    const int bx = rx == 1 ? (lx >> 2) : (rx == 0 ? 1 : 0), by = ry == 1 ? (ly >> 2) : (ry == 0 ? 1 : 0), bz = rz == 1 ? (lz >> 2) : (rz == 0 ? 1 : 0);
    int q = 0, sh = 0;
    if (rx == 1) { q |= bx << sh; ++sh; }
    if (ry == 1) { q |= by << sh; ++sh; }
    if (rz == 1) q |= bz << sh;
    const uint32_t entry = (uint32_t)(h * (27 * 5) + (rz * 9 + ry * 3 + rx) * 5);
    const uint32_t same = (uint32_t)((lz * NPT + ly) * NPT + lx);
    const uint32_t fine = (uint32_t)(((2 * lz - NPT * bz) * NPT + 2 * ly - NPT * by) * NPT + 2 * lx - NPT * bx);
    return {entry | (uint32_t)q << 9 | same << 12 | fine << 21, dst};
}
struct Items { Item at[2][27 * 64]; };
constexpr Items make_items()
{
    Items t{};
    for (int s = 0; s < 2; ++s)
        for (int n = 0; n < 27 * 64; ++n) t.at[s][n] = make_item(s != 0, n / 64, n % 64);
    return t;
}
__device__ const Items kItems = make_items();
struct PaddedItems { uint32_t at[2][27 * 64]; };
constexpr PaddedItems make_padded_items()
{
    PaddedItems t{};
    for (int s = 0; s < 2; ++s)
        for (int n = 0; n < 27 * 64; ++n) t.at[s][n] = padded_source(s != 0, ghost_item(n / 64, n % 64));
    return t;
}
__device__ const PaddedItems kPaddedItems = make_padded_items();
constexpr bool padded_items_inside()
{
    const PaddedItems t = make_padded_items();
    for (int s = 0; s < 2; ++s)
        for (int n = 0; n < 27 * 64; ++n)
            if (t.at[s][n] + 2 > (s ? 1u : 2u) * PBLK) return false;
    return true;
}
static_assert(padded_items_inside(), "every pair lies in the unit's padded blocks");

__device__ __forceinline__ Pair fma2(Pair a, Pair b, Pair c) { return Pair{fma(a.x, b.x, c.x), fma(a.y, b.y, c.y)}; }
__device__ __forceinline__ Pair fma2(double a, Pair b, Pair c) { return Pair{fma(a, b.x, c.x), fma(a, b.y, c.y)}; }

template <bool NT_>
__device__ __forceinline__ Pair ldp(const double* base, uint32_t off)
{
    asm volatile("" : "+v"(off));
    const PairAt8* p = reinterpret_cast<const PairAt8*>(reinterpret_cast<const char*>(base) + off);
    return NT_ ? (Pair)__builtin_nontemporal_load(p) : (Pair)*p;
}
template <bool NT_>
__device__ __forceinline__ void stp(double* base, uint32_t off, Pair v)
{
    asm volatile("" : "+v"(off));
    PairAt8* p = reinterpret_cast<PairAt8*>(reinterpret_cast<char*>(base) + off);
    if (NT_) __builtin_nontemporal_store(v, p); else *p = v;
}
__device__ __forceinline__ Pair lds2(const double* p) { return *reinterpret_cast<const Pair*>(p); }
__device__ __forceinline__ void lds2(double* p, Pair v) { *reinterpret_cast<Pair*>(p) = v; }

// Sources as in source.hpp; bit 1 of one in the zipped array says that the neighbour is finer, so that the second value of a
// pair lies 16 bytes further instead of 8
constexpr uint32_t kFinerBit = 2;

// what is computed so far is computed here: the compiler would move it behind the stores to LDS that follow, which wait for loads
__device__ __forceinline__ void pin(Pair& v)
{
    asm volatile("" : "+v"(v));
    __builtin_amdgcn_sched_barrier(0);
}

struct Taps { Pair m3, m2, m1, p1, p2, p3; };
// along x, own = the pair itself, t points at its first value
__device__ __forceinline__ Taps x_taps(const double* t, Pair own)
{
    const double a = t[-3], d = t[4];
    const Pair b = lds2(t - 2), c = lds2(t + 2);
    return {Pair{a, b.x}, b, Pair{b.y, own.x}, Pair{own.y, c.x}, c, Pair{c.y, d}};
}
template <int ST>
__device__ __forceinline__ Taps taps(const double* t)
{
    return {lds2(t - 3 * ST), lds2(t - 2 * ST), lds2(t - ST), lds2(t + ST), lds2(t + 2 * ST), lds2(t + 3 * ST)};
}
// Factors that are powers of two are moved through roundings, which changes no result (short of underflow): scale1 = C60 / h for
// (t * C60) * ih, scale2 = 2 C180 / h^2 for the second derivative of half the sum.
__device__ __forceinline__ Pair d1(const Taps& a, double scale1)
{
    const Pair e1 = a.p1 - a.m1, e2 = a.p2 - a.m2, e3 = a.p3 - a.m3;
    return fma2(45.0, e1, fma2(-9.0, e2, e3)) * scale1;
}
__device__ __forceinline__ double d1_single(double m3, double m2, double m1, double p1, double p2, double p3, double scale1)
{
    return fma(45.0, p1 - m1, fma(-9.0, p2 - m2, p3 - m3)) * scale1;
}
struct Axis { Pair d1, d2, ko; };
template <bool WITH_D2>
__device__ __forceinline__ Axis axis(const Taps& a, Pair u0, double scale1, double scale2)
{
    Axis r;
    r.d1 = d1(a, scale1);
    const Pair s1 = a.p1 + a.m1, s2 = a.p2 + a.m2, s3 = a.p3 + a.m3;
    r.ko = fma2(-20.0, u0, fma2(15.0, s1, fma2(-6.0, s2, s3)));
    r.d2 = WITH_D2 ? fma2(-245.0, u0, fma2(135.0, s1, fma2(-13.5, s2, s3))) * scale2 : Pair{0.0, 0.0};
    return r;
}

// Indexes of a thread into the arrays in LDS.  Everything is reached from these by constant offsets; fresh() keeps the compiler from
// working out, for every such offset that an instruction cannot hold, a register of its own for the whole kernel.
struct Place {
    int own;             // the thread's points in the D1_z array; 3 PS more in a tile (offsets in LDS instructions are not negative)
    int owny;            // in the D1_y array
    int pair;            // 2 tid
    int row, col, colto; // lowest taps and destinations (in the D1 arrays) of the ghost positions of D1
    int dst[ITEMS];
};
__device__ __forceinline__ void fresh(Place& p)
{
    asm volatile("" : "+v"(p.own), "+v"(p.owny), "+v"(p.pair), "+v"(p.row), "+v"(p.col), "+v"(p.colto));
#pragma unroll
    for (int m = 0; m < ITEMS; ++m) asm volatile("" : "+v"(p.dst[m]));
}

// D1 at the ghost positions that the outer operators of the mixed derivatives read, in pairs: each wavefront takes one of four pairs of
// x columns (positions 0..3 and 20..23 of a row: the outermost are padding, their values are never read) and one of the two
// operators, lanes are points (j, k); the first six also D1_z of a ghost y row, lanes are eight pairs of eight planes.
__device__ __forceinline__ void mixed_fill_places(Place& p, int w, int lane)
{
    const int j = (lane & 3) | ((lane >> 3) & 4), k = (lane >> 2) & 7, x = 2 * (w & 1) + (w & 2 ? 2 * NPT + PAD + X0 : 0);
    const bool along_z = w < 4;                      // uniform
    p.row = at(lane >> 3, gyz(w < 6 ? w : 0), PAD + 2 * (lane & 7));
    p.col = (k + (along_z ? 0 : PAD)) * PS + (j + (along_z ? PAD : 0)) * RS + x;         // the lowest tap
    p.colto = along_z ? k * PS + (j + PAD) * RS + x : WZ + k * YPS + j * RS + x;
}

// a value that is the same for all lanes, in scalar registers
__device__ __forceinline__ double scalar(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    return __longlong_as_double((long long)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)b)));
}
typedef const __attribute__((address_space(1))) double* Global;
typedef const __attribute__((address_space(1))) PairAt8* GlobalPair;

// read through the constant address space: a scalar load
__device__ __forceinline__ int32_t scalar_int(const void* p) { return *(const __attribute__((address_space(4))) int32_t*)(uintptr_t)p; }

// What a wavefront's threads need to know of a unit
struct Unit {
    int64_t b0;
    uint32_t o8;             // byte offset of the thread's points in a variable's zipped array (phantom: of the same ones of the real block);
                             // padded input: this and the sources in the unit's padded blocks
    uint32_t own;            // source of the thread's own values in the tile
    uint32_t src[ITEMS];     // of its ghost items
    uint32_t phantom;        // uniform over the wavefront
    // uniform, bit m is item m, bit ITEMS the own values: some lane's values are 16 bytes apart; all lanes' lie in the zipped array
    uint32_t apart, real;
};

// EPI = kOutPadded: padded in, padded out
template <int EPI, bool NTL, bool NTS>
__device__ __forceinline__ void rhs_brick(const DeviceTree& tr, const RhsArgs& a)
{
    constexpr bool PADDED = EPI == kOutPadded;
    __shared__ __attribute__((aligned(16))) double tile[TILE];
    __shared__ __attribute__((aligned(16))) double wyz[BUF];
    __shared__ __attribute__((aligned(16))) double lapS[10 * 2 * br::NT];
    __shared__ int32_t gt[2 * 27 * 5];
    double* const wz = wyz;
    double* const wy = wyz + WZ;

    int64_t nb = tr.nb, n_virt = tr.n_virt;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = w >> 2, i = 2 * (lane & 3), j = (lane >> 2) & 7, k = 2 * (w & 3) + (lane >> 5);
    const int xi = i + NPT * half;
    Place at_;
    at_.own = at(k, j + PAD, xi + PAD);
    at_.owny = k * YPS + j * RS + xi + PAD + X0;
    at_.pair = 2 * tid;
    mixed_fill_places(at_, w, lane);
#pragma unroll
    for (int m = 0; m < ITEMS; ++m) at_.dst[m] = (int)kItems.at[0][min(m * br::NT + tid, 27 * 64 - 1)].dst;

    // the table rows of a unit's two blocks are adjacent; a single block's row twice
    auto table_row = [&](int32_t unit) -> int32_t {
        if (PADDED || tid >= 2 * 27 * 5) return 0;
        const int64_t b0 = unit & ~kUnitSingle;
        return tr.ghost_v[b0 * (27 * 5) + ((unit & kUnitSingle) && tid >= 27 * 5 ? tid - 27 * 5 : tid)];
    };
    auto make_unit = [&](Unit& n, int32_t unit) {          // the table rows are in gt
        const bool single = unit & kUnitSingle;            // uniform
        n.b0 = unit & ~kUnitSingle;
        n.phantom = single && half;
        if constexpr (PADDED) {
            const uint32_t inner = padded_index(PAD, PAD, PAD), at = (uint32_t)((k * NP + j) * NP + i);
            n.o8 = (inner + at + (half && !single ? PBLK : 0)) * 8u;
            // a phantom's first columns are the real block's ghosts beyond the upper x face
            n.own = n.phantom && i < PAD ? (inner + at + NPT) * 8u : n.o8;
            n.apart = 0;
            n.real = (2u << ITEMS) - 1;
#pragma unroll
            for (int m = 0; m < ITEMS; ++m)
                if (m < ITEMS - 1 || w < LAST_ITEM_WAVES) n.src[m] = kPaddedItems.at[single][m * br::NT + tid] * 8u;
            return;
        }
        n.o8 = ((uint32_t)(n.b0 + (single ? 0 : half)) * BLK + (k * NPT + j) * NPT + i) * 8u;
        n.own = n.o8;
        n.apart = 0;
        n.real = n.phantom ? 0 : 1u << ITEMS;
        auto pick = [&](int entry, int ch, uint32_t same, uint32_t fine, bool fixed, int m) -> uint32_t {
            const int32_t* e = &gt[entry];
            const int kind = e[0];
            const bool finer = kind == K_FINER && !fixed, virt = kind == K_VIRT && !fixed;
            const uint32_t id = fixed ? (uint32_t)n.b0 : (uint32_t)e[1 + (finer ? ch : 0)];
            uint32_t s = (id * BLK + (fixed ? 0 : finer ? fine : same)) * 8u;
            if (virt) s |= 1u;
            if (finer) s |= kFinerBit;
            if (__builtin_amdgcn_ballot_w64(finer)) n.apart |= 1u << m;
            if (__builtin_amdgcn_ballot_w64(virt) == 0) n.real |= 1u << m;
            return s;
        };
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) {
            if (m == ITEMS - 1 && w >= LAST_ITEM_WAVES) continue;          // uniform
            const uint32_t it = kItems.at[single][m * br::NT + tid].where;
            n.src[m] = pick(it & 0x1ff, (it >> 9) & 3, (it >> 12) & 0x1ff, (it >> 21) & 0x1ff, it & kFixed, m);
        }
        if (n.phantom)                                     // its first columns are the real block's ghosts beyond the upper x face
            n.own = pick(14 * 5, (j >> 2) | (k >> 2) << 1, (k * NPT + j) * NPT + i, ((2 * (k & 3)) * NPT + 2 * (j & 3)) * NPT + 2 * i,
                         xi - NPT >= PAD, ITEMS);
    };

    // where the offsets of points start, variable v, unit at block b0
    auto start = [&](int64_t b0, int v) -> int64_t { return PADDED ? ((int64_t)v * nb + b0) * PBLK : (int64_t)v * nb * BLK; };
    // No branch does anything but load to a register that another load may have written: the compiler would wait for the loads where
    // such branches join.
    struct Fetch { Pair own, g[ITEMS]; double own2, g2[ITEMS]; };          // second values 16 bytes apart come by themselves
    auto request = [&](Fetch& f, const Unit& n, int v, auto first, auto last) {      // items first .. last - 1, -1: own values
        constexpr int FIRST = decltype(first)::value, LAST = decltype(last)::value;
        const double* base = a.in + start(n.b0, v);
        const double* vbase = a.virt + (int64_t)v * n_virt * BLK;
        auto load = [&](Pair& to, double& to2, uint32_t s, int m) {
            if (PADDED || (n.real >> m & 1)) {             // uniform
                to = ldp<false>(base, s & ~7u);
            } else {
                asm volatile("" : "+v"(s));          // or lane masks for every item would be kept
                const bool virt = s & 1u;
                to = *(GlobalPair)((uint64_t)(uintptr_t)(virt ? vbase : base) + (s & ~7u));
            }
            if (n.apart >> m & 1) {                        // uniform
                asm volatile("" : "+v"(s));
                if ((s & 3u) == kFinerBit) to2 = *(Global)((uint64_t)(uintptr_t)base + (s & ~7u) + 16);
            }
        };
        if (FIRST < 0) load(f.own, f.own2, n.own, ITEMS);
#pragma unroll
        for (int m = FIRST < 0 ? 0 : FIRST; m < LAST; ++m)
            if (m < ITEMS - 1 || w < LAST_ITEM_WAVES) load(f.g[m], f.g2[m], n.src[m], m);
    };
    using N1 = std::integral_constant<int, -1>;
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    using P4 = std::integral_constant<int, ITEMS>;
    auto prefetch = [&](Fetch& f, const Unit& n, int v, auto edges) {
        request(f, n, v, N1{}, std::integral_constant<int, decltype(edges)::value ? ITEMS : FACE_ITEMS>{});
    };
    auto commit = [&](double* to, Fetch& f, const Unit& n, auto edges) -> Pair {
        constexpr bool EDGES = decltype(edges)::value;
        auto finish = [&](Pair& v, double v2, uint32_t s, int m) {
            if (!PADDED && (n.apart >> m & 1)) {     // uniform
                asm volatile("" : "+v"(s));
                v.y = (s & 3u) == kFinerBit ? v2 : v.y;
            }
        };
        finish(f.own, f.own2, n.own, ITEMS);
        lds2(&to[at_.own + PAD * PS], f.own);
#pragma unroll
        for (int m = 0; m < (EDGES ? ITEMS : FACE_ITEMS); ++m)
            if (m < ITEMS - 1 || w < LAST_ITEM_WAVES) {
                finish(f.g[m], f.g2[m], n.src[m], m);
                lds2(&to[at_.dst[m]], f.g[m]);
            }
        return f.own;
    };
    using Edges = std::true_type;
    using Faces = std::false_type;
    auto fence = []() { __builtin_amdgcn_sched_barrier(0); };

    const int wg = blockIdx.x % kRound;
    const Rounds mine = rounds_of_part(blockIdx.x / kRound, gridDim.x / kRound, rounds_of(tr.n_units));
    int64_t round = mine.first, q = round < mine.last ? unit_of_round(round, wg, tr.n_units) : -1;
    if (q < 0) return;                               // uniform
    int32_t unit = scalar_int(&tr.units[q]);
    if (!PADDED) {
        if (tid < 2 * 27 * 5) gt[tid] = table_row(unit);
        __syncthreads();
    }
    Unit me;
    make_unit(me, unit);

    auto centre = [&](const Unit& n, int v) -> Pair { return ldp<false>(a.in + start(n.b0, v), n.o8); };
    struct Epi { Pair acc, u; };
    auto epi_load = [&](Epi& e, int f) {
        if (EPI == kRkMiddle || EPI == kRkLast) {
            const int64_t o = (int64_t)f * nb * BLK;
            e.u = ldp<NTL>(a.u + o, me.o8);
            e.acc = ldp<NTL>(a.acc + o, me.o8);
        }
    };
    // the right-hand side, or accumulator and stage vector, or the new state
    struct Result { Pair a, b; };
    auto result = [&](Pair r, const Epi& e, Pair own) -> Result {
        Result o{r, r};
        if (EPI == kRkFirst) o.b = fma2(a.c, r, own);
        else if (EPI == kRkMiddle) o = {fma2(2.0, r, e.acc), fma2(a.c, r, e.u)};
        else if (EPI == kRkLast) o.a = fma2(a.c, e.acc + r, e.u);
        pin(o.a);
        if (EPI == kRkFirst || EPI == kRkMiddle) pin(o.b);
        return o;
    };
    auto put = [&](int f, const Result& r) {
        if (me.phantom) return;                      // uniform
        const int64_t o = (int64_t)f * nb * BLK;
        if (PADDED) stp<NTS>(a.out + start(me.b0, f), me.o8, r.a);
        else if (EPI == kOutZipped) stp<NTS>(a.out + o, me.o8, r.a);
        else if (EPI == kRkLast) stp<NTS>(a.u + o, me.o8, r.a);
        else { stp<NTS>(a.acc + o, me.o8, r.a); stp<NTS>(a.out + o, me.o8, r.b); }
    };

    Fetch F, H;
    Epi e, e1;
    prefetch(F, me, syn24_stream(0), Faces{});
    prefetch(H, me, syn24_stream(1), Edges{});
    Pair u0 = centre(me, 0), bx = centre(me, 1), by = centre(me, 2), bz = centre(me, 3);
    Pair u4 = centre(me, 4), u5 = centre(me, 5), u6 = centre(me, 6), u7 = centre(me, 7), u8 = centre(me, 8), u9 = centre(me, 9);
    Pair own = commit(tile, F, me, Faces{});
    __syncthreads();
#pragma unroll 1
    for (;;) {
    asm volatile("" : "+s"(nb), "+s"(n_virt));       // or the addresses of all variables in all arrays would be kept from unit to unit
    // the tile of variable 10 is complete, the data of variable 9 is on its way
    const int lvl = scalar_int(&tr.leaves[me.b0].level);
    const double ih = __longlong_as_double((long long)(1026 + lvl) << 52), ih2 = __longlong_as_double((long long)(1029 + 2 * lvl) << 52);
    const double scale1 = scalar(C60 * ih), scale2 = scalar((2.0 * C180) * ih2), scale_ko = scalar(a.sigma * over64(ih));
    q = ++round < mine.last ? unit_of_round(round, wg, tr.n_units) : -1;
    const bool more = q >= 0;                        // uniform
    if (more) unit = scalar_int(&tr.units[q]);
    const int32_t row = more ? table_row(unit) : 0;
    // G_dd = 1 - u / 8 is worked out where it is used, G_de = -u / 8 goes into a factor
    auto diagonal = [](Pair u) -> Pair { return fma2(-0.125, u, Pair{1.0, 1.0}); };
    Pair nx, ny, nz;

    auto tx = [&](const double* T) -> Taps { return x_taps(T + (at_.own + PAD * PS), own); };
    auto ty = [&](const double* T) -> Taps { return taps<RS>(T + (at_.own + PAD * PS)); };
    auto tz = [&](const double* T) -> Taps { return taps<PS>(T + (at_.own + PAD * PS)); };
    // what a pass computes before the second derivatives join, as syn24_axes()
    struct Part { Pair t1, t3q, ko, diag; };
    auto axes = [&](const double* T, auto with_d2, auto after_x, auto after_y) -> Part {
        constexpr bool D2 = decltype(with_d2)::value;
        Part r;
        r.diag = Pair{0.0, 0.0};
        const Axis x = axis<D2>(tx(T), own, scale1, scale2);
        r.t1 = bx * x.d1;
        r.t3q = x.d1 * nx;
        nx = x.d1;
        if (D2) r.diag = diagonal(u4) * x.d2;
        Pair ks = x.ko;
        fence();
        after_x();
        fence();
        const Axis y = axis<D2>(ty(T), own, scale1, scale2);
        r.t1 = fma2(by, y.d1, r.t1);
        r.t3q = fma2(y.d1, ny, r.t3q);
        ny = y.d1;
        if (D2) { r.diag = fma2(diagonal(u7), y.d2, r.diag); lds2(&wy[at_.owny], y.d1); }
        ks = ks + y.ko;
        fence();
        after_y();
        fence();
        const Axis z = axis<D2>(tz(T), own, scale1, scale2);
        r.t1 = fma2(bz, z.d1, r.t1);
        r.t3q = fma2(z.d1, nz, r.t3q);
        nz = z.d1;
        if (D2) { r.diag = fma2(diagonal(u9), z.d2, r.diag); lds2(&wz[at_.own], z.d1); }
        r.ko = scale_ko * (ks + z.ko);
        return r;
    };
    auto combine = [&](const Part& p, int f, Pair lap, Pair unext) -> Pair {
        const double kappa = __longlong_as_double((long long)(1023 - (f & 3)) << 52);
        return fma2(-0.5, u0 * unext, fma2(0.25, p.t3q, fma2(kappa, lap, p.t1))) + p.ko;
    };
    const int col_step = w < 4 ? PS : RS;            // uniform

    // pass 0: gradient of variable 10 only
    const Pair u10 = own;
    nx = d1(tx(tile), scale1); ny = d1(ty(tile), scale1); nz = d1(tz(tile), scale1);
    pin(nx); pin(ny); pin(nz);
    __syncthreads();                                 // everybody is done with the tile
    own = commit(tile, H, me, Edges{});
    __syncthreads();
    auto pass_d2 = [&](int t, auto next_edges) {
        const int f = syn24_stream(t);
        fresh(at_);
        const Pair unext = centre(me, (f + 11) % 24);
        epi_load(e, f);
        const double* tc = tile + at_.col;
        const Taps C{lds2(tc), lds2(tc + col_step), lds2(tc + 2 * col_step), lds2(tc + 4 * col_step), lds2(tc + 5 * col_step), lds2(tc + 6 * col_step)};
        lds2(&wyz[at_.colto], d1(C, scale1));
        if (w < 6) lds2(&wz[at_.row], d1(taps<PS>(tile + (at_.row + PAD * PS)), scale1));          // uniform
        fence();
        request(F, me, syn24_stream(t + 1), N1{}, P1{});
        fence();
        Part p = axes(tile, std::true_type{}, [&] { request(F, me, syn24_stream(t + 1), P1{}, P2{}); },
                      [&] { if (decltype(next_edges)::value) request(F, me, syn24_stream(t + 1), P2{}, P4{}); });
        asm volatile("" : "+v"(p.t1), "+v"(p.t3q), "+v"(p.ko), "+v"(p.diag));   // not behind the barrier, with all their operands alive
        __syncthreads();
        fresh(at_);
        const Pair dxy = d1(x_taps(wy + at_.owny, ny), scale1), dxz = d1(x_taps(wz + at_.own, nz), scale1), dyz = d1(taps<RS>(wz + at_.own), scale1);
        const Pair lap = fma2(-0.25, fma2(u8, dyz, fma2(u6, dxz, u5 * dxy)), p.diag);
        lds2(&lapS[f * 2 * br::NT + at_.pair], lap);
        const Result r = result(combine(p, f, lap, unext), e, own);
        own = commit(tile, F, me, next_edges);
        put(f, r);
        __syncthreads();                             // the tile is complete; D1_y u, D1_z u may be overwritten
    };
#pragma unroll 1
    for (int t = 1; t < 10; ++t) pass_d2(t, Edges{});
    pass_d2(10, Faces{});
    if (!PADDED && tid < 2 * 27 * 5) gt[tid] = row;  // of the next unit; read behind the barriers of the passes that follow
    // Passes over the variables without second derivatives: the tile and the D1 arrays, now idle, in turn.  They are shorter than
    // the way to memory and back, so the data of the variable after the next one is requested.
    auto pass_light = [&](double* T, double* next, int t, Pair unext, Fetch& coming, Fetch& after, Epi& now, Epi& then) {
        const int f = syn24_stream(t);
        fresh(at_);
        const Pair lap = lds2(&lapS[(f % 10) * 2 * br::NT + at_.pair]);
        const Part p = axes(T, std::false_type{},
                            [&] { if (t + 1 < NSTREAM) epi_load(then, syn24_stream(t + 1)); if (t + 2 < NSTREAM) request(after, me, syn24_stream(t + 2), N1{}, P0{}); },
                            [&] { if (t + 2 < NSTREAM) request(after, me, syn24_stream(t + 2), P0{}, P2{}); });
        const Result r = result(combine(p, f, lap, unext), now, own);
        if (t + 1 < NSTREAM) own = commit(next, coming, me, Faces{});
        put(f, r);
        if (t + 1 < NSTREAM) __syncthreads();
    };
    // u_{a+11}: a = 23..13 -> u_10..u_0, a = 12, 11, 10 -> u_23, u_22, u_21
    prefetch(H, me, syn24_stream(12), Faces{});
    epi_load(e, syn24_stream(11));
    const Pair u23 = own;
    pass_light(tile, wyz, 11, u10, H, F, e, e1);
    const Pair u22 = own;
    pass_light(wyz, tile, 12, u9, F, H, e1, e);
    const Pair u21 = own;
    pass_light(tile, wyz, 13, u8, H, F, e, e1);
    pass_light(wyz, tile, 14, u7, F, H, e1, e);
    pass_light(tile, wyz, 15, u6, H, F, e, e1);
    pass_light(wyz, tile, 16, u5, F, H, e1, e);
    pass_light(tile, wyz, 17, u4, H, F, e, e1);
    pass_light(wyz, tile, 18, bz, F, H, e1, e);
    pass_light(tile, wyz, 19, by, H, F, e, e1);
    pass_light(wyz, tile, 20, bx, F, H, e1, e);
    pass_light(tile, wyz, 21, u0, H, F, e, e1);
    pass_light(wyz, tile, 22, u23, F, H, e1, e);
    // the data of the first variables of the next unit is requested two passes ahead too
    Unit next{};
    if (more) {
        make_unit(next, unit);
        prefetch(F, next, syn24_stream(0), Faces{});
        u4 = centre(next, 4); u5 = centre(next, 5); u6 = centre(next, 6); u7 = centre(next, 7); u8 = centre(next, 8); u9 = centre(next, 9);
    }
    pass_light(tile, wyz, 23, u22, H, F, e, e1);
    if (more) prefetch(H, next, syn24_stream(1), Edges{});
    pass_light(wyz, tile, 24, u21, F, H, e1, e);
    if (!more) break;
    own = commit(tile, F, next, Faces{});
    me.b0 = next.b0; me.o8 = next.o8; me.own = next.own; me.phantom = next.phantom; me.apart = next.apart; me.real = next.real;
#pragma unroll
    for (int m = 0; m < ITEMS; ++m) me.src[m] = next.src[m];
    u0 = centre(me, 0); bx = centre(me, 1); by = centre(me, 2); bz = centre(me, 3);
    __syncthreads();
    }
}

}  // namespace br

template <int EPI, bool NTL, bool NTS>
__global__ __launch_bounds__(br::NT) void k_brick(DeviceTree tr, RhsArgs a) { br::rhs_brick<EPI, NTL, NTS>(tr, a); }

// Padded in, padded out.  What bounds it is memory traffic.  Of the ghosts of the input the faces of all variables are read and the edges of fields 0..9,
// but no corners and none between the two blocks; of the own values those of fields 0..20 twice (0..9 also as pointwise factors, 10 as the first and
// the last of the stream, 11..20 also as u_{a+11}), the second time mostly from the caches.  Only the 8^3 interior of an output block is
// written, 64 bytes of every 112, so that no line of it is whole.  Plain stores wait in the L2 for the rest of a line and are then
// completed from memory all the same; non-temporal ones push nothing else out.  Rows start at any multiple of 8 bytes, which is all that
// the accesses ask for, and the sources are the same for all units.
// (us, one block per workgroup, a thread per point, Lap parked in the output -> as here with plain stores -> as here: 512 blocks 88 -> 68 -> 62,
// 792 179 -> 146 -> 117, 5,230 1135 -> 1034 -> 839, 21,064 4510 -> 4198 -> 3436; the pipeline of unzip, this and zip 207 -> 191 -> 193,
// 384 -> 341 -> 334, 2473 -> 2363 -> 2184, 9678 -> 9334 -> 8590.)
__global__ __launch_bounds__(br::NT) void k_brick_padded(DeviceTree tr, RhsArgs a) { br::rhs_brick<kOutPadded, false, true>(tr, a); }

inline dim3 grid_for_units(int64_t n_units) { return dim3(kRound * (unsigned)parts_of(rounds_of(n_units))); }

// Operands of a stage are read non-temporally from the size at which a step's four vectors fill the 256 MB memory-side cache, us without / with: 196 / 203 on 512
// blocks (201 MB), 357 / 366 on 575 (226 MB), 388 / 400 on 631 (248 MB), 421 / 418 on 694 (272 MB), 464 / 448 on 778 (305 MB); with
// the centred rule 374 / 383, 419 / 429, 448 / 445, 505 / 486 on the last four.
constexpr int64_t kOperandStepBytes = 256ll << 20;

template <int EPI>
void launch_bricks(const DeviceTree& t, const RhsArgs& a, hipStream_t s)
{
    const dim3 grid = grid_for_units(t.n_units), block(br::NT);
    constexpr bool kOperands = EPI == kRkMiddle || EPI == kRkLast;
    // Written non-temporally from the sizes that kernels.hpp explains, us without / with (operands past the caches on both sides): steps 448 / 453 on
    // 764 blocks (300 MB), 457 / 453 on 792, 462 / 463 on 834 (327 MB), 483 / 467 on 890 (349 MB), 521 / 508 on 981, 723 / 684 on 1,198;
    // with the centred rule 485 / 492, 494 / 496, 499 / 509, 527 / 521, 576 / 577, 785 / 754.
    const int64_t bytes = t.nb * BLK * (int64_t)sizeof(double) * 24 * (EPI == kOutZipped ? 2 : 4);
    const bool stream = bytes > (EPI == kOutZipped ? kStreamEvalBytes : kStreamStepBytes);
    if (stream) hipLaunchKernelGGL((k_brick<EPI, kOperands, true>), grid, block, 0, s, t, a);
    else if (kOperands && bytes > kOperandStepBytes) hipLaunchKernelGGL((k_brick<EPI, kOperands, false>), grid, block, 0, s, t, a);
    else hipLaunchKernelGGL((k_brick<EPI, false, false>), grid, block, 0, s, t, a);
}

}  // namespace

hipError_t launch_rhs_bricks(const DeviceTree& t, Epilogue ep, const RhsArgs& a, hipStream_t s)
{
    if (ep != kOutPadded && t.n_virt > kBlockLimit) return hipErrorInvalidValue;     // sources here are of 32 bits
    switch (ep) {
    case kOutPadded: hipLaunchKernelGGL(k_brick_padded, grid_for_units(t.n_units), dim3(br::NT), 0, s, t, a); break;
    case kOutZipped: launch_bricks<kOutZipped>(t, a, s); break;
    case kRkFirst: launch_bricks<kRkFirst>(t, a, s); break;
    case kRkMiddle: launch_bricks<kRkMiddle>(t, a, s); break;
    case kRkLast: launch_bricks<kRkLast>(t, a, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace octfd
