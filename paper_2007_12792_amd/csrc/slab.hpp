// Right-hand side of the kinds with one or two variables (DERIVS, WAVE, BURGERS): a wavefront owns a slab of two z planes
// of one block and one variable.  Private to kernels.hip.
//
// These kernels do little arithmetic per byte, and what holds them is how much of the memory traffic is in flight:
//   - lanes are the 64 points (i, j) of a plane.  A wavefront requests its two own planes (512 bytes each), the 3 x 8 x 2
//     ghost values beyond each x and y face (one load each, lanes 0..47) and one or two of the six ghost planes: eight loads
//     a lane at most, all issued before the first is waited for, with up to 32 wavefronts on a compute unit;
//   - every value is requested once per block.  (A first version without any exchange between the wavefronts of a block,
//     where each loaded all eight planes of its columns, was no faster than one thread per point: the L1 stalls on a
//     request for a line that is still on its way, half of the kernel's time by its counter.)  The values meet in LDS
//     behind the one barrier;
//     (Step of the wave system / Burgers on 47,783 blocks: 1645 / 789 us, 1501 / 705 us with the non-temporal accesses of
//     k_rhs_stream; 1730 / 970 us with one thread per point and a fill plan; 1802 / 833 us without the exchange.)
//   - which octant lies beyond a face is the same for all lanes, so the table row is read with scalar loads that are issued
//     together, the base address of a load is scalar, and a finer neighbour is a uniform branch without loads in it.
#pragma once
#include "stencils.hpp"

namespace octfd {
namespace {

namespace sl {
constexpr int KZ = 2, NSLAB = NPT / KZ;              // planes per slab, slabs per block
constexpr int NZ = KZ + 2 * PAD;                     // planes of a lane's column
constexpr int XRS = 24;                              // stride of the 14-point x rows: 8 * odd, so that four rows of eight points
                                                     // fall into 32 different 8-byte banks (28, the next even fit, costs 2-way conflicts)
constexpr int YG = NPT * XRS;                        // the y ghost rows (three below, three above) of eight points behind the x rows
constexpr int PLANE = YG + 2 * PAD * NPT;            // 240
constexpr int NGL = PAD * NPT * KZ;                  // ghost values beyond one x or y face: 48
constexpr int ZG = NPT * PLANE;                      // the six z ghost planes of 64 points behind the eight planes
constexpr int LDS = ZG + 2 * PAD * 64;               // per block and variable, in doubles (18 KB)
}  // namespace sl

constexpr int kDirXm = 12, kDirXp = 14, kDirYm = 10, kDirYp = 16, kDirZm = 4, kDirZp = 22;   // table entries of the six faces

struct Slab {
    double own[sl::KZ];                              // planes k0, k0+1 at (i, j)
    double zg[2];                                    // ghost planes zg0, zg0+1 (the second in the outer slabs only)
    double g[4];                                     // lanes 0..47: ghost value beyond the faces x-, x+, y-, y+
};
// the six ghost planes -3, -2, -1, 8, 9, 10 are numbers 0..5; slab w loads {0, 1}, {2}, {3}, {4, 5}
__device__ __forceinline__ int first_ghost_plane(int w) { return w + (w > 0 ? 1 : 0); }
__device__ __forceinline__ bool two_ghost_planes(int w) { return w == 0 || w == 3; }

// lane -> its value beyond an x face (column c of three, row j, plane k0 + k) or a y face (row c, point i, plane k0 + k)
struct GhostLane { int xc, xj, xk, yc, yi, yk; };
__device__ __forceinline__ GhostLane ghost_lane(int lane)
{
    const int l = min(lane, sl::NGL - 1), r = l / PAD, t = l >> 3;   // the lanes past 47 repeat the last value
    return {l - PAD * r, r & 7, r >> 3, t % PAD, l & 7, t / PAD};
}

// Table entries are read through the constant address space: scalar loads, all of them issued before the first is needed.
typedef const __attribute__((address_space(4))) int32_t* ScalarInts;
__device__ __forceinline__ ScalarInts scalar_ints(const void* p) { return (ScalarInts)(uintptr_t)p; }

// the octant beyond a face: base of the array that holds it (of virtual blocks: of the 4 GiB of it), and byte offset of the
// lane's value from there, modulo 2^32 like a source
struct FaceEntry { int kind, id[4]; };
__device__ __forceinline__ FaceEntry face_entry(ScalarInts row, int dir)
{
    ScalarInts e = row + dir * 5;
    return {e[0], {e[1], e[2], e[3], e[4]}};
}
// same: index of the value in a block of the same level (real or virtual); in a subdivided octant q = which of the face's
// four children holds the point, fine = index of the coinciding node.  No loads here, so nothing waits on the branch.
__device__ __forceinline__ uint32_t face_offset(const FaceEntry& e, int q, int fine, int same)
{
    if (e.kind != K_FINER) return ((uint32_t)e.id[0] * BLK + same) * 8u;   // uniform
    const int32_t id = q == 0 ? e.id[0] : (q == 1 ? e.id[1] : (q == 2 ? e.id[2] : e.id[3]));
    return ((uint32_t)id * BLK + fine) * 8u;
}

// slab w of block b, zipped input: `in`, `virt` are the variable's arrays, `row` the block's table row
__device__ __forceinline__ void load_slab_zipped(Slab& s, ScalarInts row, const double* in, const double* virt, int64_t b, int w, int lane,
                                                 const GhostLane& gl)
{
    const int i = lane & 7, j = lane >> 3, k0 = sl::KZ * w, khalf = k0 >> 2;
    // the two lower slabs reach below the block, the two upper ones above it
    const FaceEntry ez = face_entry(row, w < 2 ? kDirZm : kDirZp);
    const FaceEntry e0 = face_entry(row, kDirXm), e1 = face_entry(row, kDirXp), e2 = face_entry(row, kDirYm), e3 = face_entry(row, kDirYp);
    auto base = [&](const FaceEntry& e) -> const double* { return e.kind == K_VIRT ? virt + bank_start(e.id[0]) : in; };
    const uint32_t o = ((uint32_t)b * BLK + k0 * 64 + lane) * 8u;
#pragma unroll
    for (int kk = 0; kk < sl::KZ; ++kk) s.own[kk] = ldg(in + kk * 64, o);
    const uint32_t zoff = face_offset(ez, (i >> 2) | (j >> 2) << 1, 2 * (j & 3) * NPT + 2 * (i & 3), lane);
    const int lz = w < 2 ? 5 + first_ghost_plane(w) : first_ghost_plane(w) - 3;      // plane in the octant beyond the face
    const int zstep = ez.kind == K_FINER ? 2 * 64 : 64, z0 = (ez.kind == K_FINER ? lz & 3 : lz) * zstep;
    s.zg[0] = ldg(base(ez) + z0, zoff);
    if (two_ghost_planes(w)) s.zg[1] = ldg(base(ez) + z0 + zstep, zoff);             // uniform
    const int xk = k0 + gl.xk, yk = k0 + gl.yk;
    const int xq = (gl.xj >> 2) | khalf << 1, yq = (gl.yi >> 2) | khalf << 1;
    const int xf = (2 * (xk & 3) * NPT + 2 * (gl.xj & 3)) * NPT, xs = (xk * NPT + gl.xj) * NPT;
    const int yf = 2 * (yk & 3) * NPT * NPT + 2 * (gl.yi & 3), ys = yk * NPT * NPT + gl.yi;
    s.g[0] = ldg(base(e0), face_offset(e0, xq, xf + 2 * (gl.xc + 1), xs + gl.xc + 5));
    s.g[1] = ldg(base(e1), face_offset(e1, xq, xf + 2 * gl.xc, xs + gl.xc));
    s.g[2] = ldg(base(e2), face_offset(e2, yq, yf + 2 * (gl.yc + 1) * NPT, ys + (gl.yc + 5) * NPT));
    s.g[3] = ldg(base(e3), face_offset(e3, yq, yf + 2 * gl.yc * NPT, ys + gl.yc * NPT));
}

// the same from a padded block
__device__ __forceinline__ void load_slab_padded(Slab& s, const double* block, int w, int lane, const GhostLane& gl)
{
    const int i = lane & 7, j = lane >> 3, k0 = sl::KZ * w;
    auto at = [&](int kk, int jj, int ii) -> double { return ldg(block, ((kk * NP + jj) * NP + ii) * 8u); };
#pragma unroll
    for (int kk = 0; kk < sl::KZ; ++kk) s.own[kk] = at(k0 + kk + PAD, j + PAD, i + PAD);
    const int g = first_ghost_plane(w), z0 = w < 2 ? g : g + NPT;                    // 0..2, 11..13
    s.zg[0] = at(z0, j + PAD, i + PAD);
    if (two_ghost_planes(w)) s.zg[1] = at(z0 + 1, j + PAD, i + PAD);
    s.g[0] = at(k0 + gl.xk + PAD, gl.xj + PAD, gl.xc);
    s.g[1] = at(k0 + gl.xk + PAD, gl.xj + PAD, gl.xc + PAD + NPT);
    s.g[2] = at(k0 + gl.yk + PAD, gl.yc, gl.yi + PAD);
    s.g[3] = at(k0 + gl.yk + PAD, gl.yc + PAD + NPT, gl.yi + PAD);
}

// into the LDS of the block and variable; ends without a barrier
__device__ __forceinline__ void store_slab(double* T, const Slab& s, int w, int lane, const GhostLane& gl)
{
    const int i = lane & 7, j = lane >> 3;
    double* P = T + sl::KZ * w * sl::PLANE;
#pragma unroll
    for (int kk = 0; kk < sl::KZ; ++kk) P[kk * sl::PLANE + j * sl::XRS + PAD + i] = s.own[kk];
    double* Z = T + sl::ZG + first_ghost_plane(w) * 64 + lane;
    Z[0] = s.zg[0];
    if (two_ghost_planes(w)) Z[64] = s.zg[1];
    if (lane < sl::NGL) {
        double* x = P + gl.xk * sl::PLANE + gl.xj * sl::XRS + gl.xc;
        x[0] = s.g[0];
        x[PAD + NPT] = s.g[1];
        double* y = P + gl.yk * sl::PLANE + sl::YG + gl.yc * NPT + gl.yi;
        y[0] = s.g[2];
        y[PAD * NPT] = s.g[3];
    }
}

// the planes k0-3 .. k0+4 at (i, j): all that the z stencils of the slab read
__device__ __forceinline__ void load_column(double (&z)[sl::NZ], const double* T, const Slab& s, int w, int lane)
{
    const int own = (lane >> 3) * sl::XRS + PAD + (lane & 7), k0 = sl::KZ * w;
#pragma unroll
    for (int m = 0; m < sl::NZ; ++m) {
        const int p = k0 - PAD + m;                  // uniform
        if (m >= PAD && m < PAD + sl::KZ) z[m] = s.own[m - PAD];
        else if (p >= 0 && p < NPT) z[m] = T[p * sl::PLANE + own];
        else z[m] = T[sl::ZG + (p < 0 ? p + PAD : p - NPT + PAD) * 64 + lane];
    }
}

// where in a plane the y taps j-3 .. j-1, j+1 .. j+3 of (i, j) lie: among the x rows or the ghost rows
__device__ __forceinline__ void y_taps(int (&ya)[6], int lane)
{
    const int i = lane & 7, j = lane >> 3;
#pragma unroll
    for (int m = 0; m < 6; ++m) {
        const int jj = j + (m < 3 ? m - 3 : m - 2);
        ya[m] = jj < 0 ? sl::YG + (jj + PAD) * NPT + i : (jj < NPT ? jj * sl::XRS + PAD + i : sl::YG + (jj - NPT + PAD) * NPT + i);
    }
}

// all operators at (i, j) of plane kk of the slab: the same sequences as on a tile
template <bool WITH_D2>
__device__ __forceinline__ PointOps slab_ops(const double* slab, const double (&z)[sl::NZ], const int (&ya)[6], int kk, int lane, double sigma, double ih, double ih2)
{
    const double* P = slab + kk * sl::PLANE;
    const double* X = P + (lane >> 3) * sl::XRS + PAD + (lane & 7);
    PointOps r;
    r.u0 = z[PAD + kk];
    const AxisOps x = axis_ops_taps<WITH_D2>(X[-3], X[-2], X[-1], X[1], X[2], X[3], r.u0, ih, ih2);
    const AxisOps y = axis_ops_taps<WITH_D2>(P[ya[0]], P[ya[1]], P[ya[2]], P[ya[3]], P[ya[4]], P[ya[5]], r.u0, ih, ih2);
    const AxisOps zz = axis_ops_taps<WITH_D2>(z[kk], z[kk + 1], z[kk + 2], z[kk + 4], z[kk + 5], z[kk + 6], r.u0, ih, ih2);
    r.dx = x.d1; r.dy = y.d1; r.dz = zz.d1;
    r.lap = (x.d2 + y.d2) + zz.d2;
    r.ko = sigma * (((x.ko + y.ko) + zz.ko) * over64(ih));
    return r;
}

constexpr int slab_wavefronts(int kind) { return sl::NSLAB * (kind == OT_RHS_WAVE ? 2 : 1); }

// One block per workgroup.  lds: the workgroup's LDS (sl::LDS doubles per variable); lapS: one block of doubles (WAVE
// only); NT: everything but the slabs is read and written non-temporally.
template <int KIND, bool ZIN, int EPI, bool NT>
__device__ __forceinline__ void rhs_slab(const DeviceTree& tr, const RhsArgs& a, double* lds, double* lapS, int64_t b, int tid)
{
    const int64_t nb = tr.nb;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int w = wave & (sl::NSLAB - 1), v = wave / sl::NSLAB;     // slab; variable (WAVE: u is 0, pi is 1)
    const int k0 = sl::KZ * w;
    const int lvl = *scalar_ints(&tr.leaves[b].level);
    const double ih = __longlong_as_double((long long)(1026 + lvl) << 52), ih2 = __longlong_as_double((long long)(1029 + 2 * lvl) << 52);
    const double sigma = a.sigma;
    double* T = lds + v * sl::LDS;
    const double* P = T + k0 * sl::PLANE;
    const GhostLane gl = ghost_lane(lane);
    const uint32_t o8 = ((uint32_t)b * BLK + k0 * 64 + lane) * 8u;                                    // plane k0, + 512 bytes for the next
    const uint32_t p8 = (((k0 + PAD) * NP + (lane >> 3) + PAD) * NP + (lane & 7) + PAD) * 8u;         // in a padded block, + 1568
    constexpr uint32_t OS = 64 * 8, PSB = NP * NP * 8;

    Slab s;
    if (ZIN) load_slab_zipped(s, scalar_ints(tr.ghost_v + b * (27 * 5)), a.in + v * nb * BLK, a.virt + v * tr.n_virt * BLK, b, w, lane, gl);
    else load_slab_padded(s, a.in + (v * nb + b) * PBLK, w, lane, gl);
    int ya[6];
    y_taps(ya, lane);
    double z[sl::NZ];
    if (KIND == OT_RHS_DERIVS) {
        store_slab(T, s, w, lane, gl);
        __syncthreads();
        load_column(z, T, s, w, lane);
#pragma unroll
        for (int kk = 0; kk < sl::KZ; ++kk) {
            const PointOps p = slab_ops<true>(P, z, ya, kk, lane, 0.0, ih, ih2);
            const uint32_t o = o8 + kk * OS, q = p8 + kk * PSB;
            const double val[4] = {p.dx, p.dy, p.dz, p.lap};
#pragma unroll
            for (int n = 0; n < 4; ++n) emit<EPI, NT>(a, nb, n, b, o, q, val[n], EpiOperands{0.0, 0.0});   // no stages: four outputs of one field
        }
    } else if (KIND == OT_RHS_BURGERS) {
        EpiOperands e[sl::KZ];
#pragma unroll
        for (int kk = 0; kk < sl::KZ; ++kk) e[kk] = epi_prefetch<EPI, NT>(a, nb, 0, o8 + kk * OS);
        store_slab(T, s, w, lane, gl);
        __syncthreads();
        load_column(z, T, s, w, lane);
#pragma unroll
        for (int kk = 0; kk < sl::KZ; ++kk) {
            const PointOps p = slab_ops<false>(P, z, ya, kk, lane, sigma, ih, ih2);
            const double flux = p.u0 * p.dx;
            emit<EPI, NT>(a, nb, 0, b, o8 + kk * OS, p8 + kk * PSB, p.ko - flux, with_u<EPI>(e[kk], p.u0));
        }
    } else {
        // wavefronts of u: the Laplacian goes to those of pi through LDS, d_t u = pi + KO(u) needs pi at the own points only
        EpiOperands e[sl::KZ];
        double other[sl::KZ];
#pragma unroll
        for (int kk = 0; kk < sl::KZ; ++kk) {
            e[kk] = epi_prefetch<EPI, NT>(a, nb, v, o8 + kk * OS);
            if (v == 0) other[kk] = ZIN ? ldg(a.in + nb * BLK, o8 + kk * OS) : ldg(a.in + (nb + b) * PBLK, p8 + kk * PSB);
        }
        store_slab(T, s, w, lane, gl);
        __syncthreads();
        load_column(z, T, s, w, lane);
        double ko[sl::KZ];
#pragma unroll
        for (int kk = 0; kk < sl::KZ; ++kk) {
            if (v == 0) {                            // uniform
                const PointOps p = slab_ops<true>(P, z, ya, kk, lane, sigma, ih, ih2);
                lapS[(k0 + kk) * 64 + lane] = p.lap;
                ko[kk] = p.ko;
            } else {
                ko[kk] = slab_ops<false>(P, z, ya, kk, lane, sigma, ih, ih2).ko;
            }
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < sl::KZ; ++kk) {
            const double k = v == 0 ? other[kk] + ko[kk] : lapS[(k0 + kk) * 64 + lane] + ko[kk];
            emit<EPI, NT>(a, nb, v, b, o8 + kk * OS, p8 + kk * PSB, k, with_u<EPI>(e[kk], s.own[kk]));
        }
    }
}

}  // namespace
}  // namespace octfd
