// kct_gather.h -- the pieces of the brick-gather backprojector (A^T, Section 2,
// Eq. 2), written as plain functions so the kernel is a short sequence of
// calls between barriers.
//
// A workgroup owns a brick of BX x BY x TZ voxels; each of its 256 lanes owns
// one (x, y) position and the TZ voxels above it.  For every view the
// workgroup
//   1. bounds the brick's shadow on the detector (the eight projected corners),
//   2. stages, for every pixel of the shadow, the ray's z-parameters and its
//      value multiplied by the ray length factor L in LDS (one record per
//      pixel), and the per-column in-plane ray parameters,
//   3. lets each lane gather: the interval of detector columns whose
//      rays can cross its voxel column, the in-plane xi-interval of each of those
//      columns (shared by the TZ voxels), per voxel the candidate rows from
//      the z-range of those rays, and for every candidate the exact weight of
//      kct_weights.h.
// The shadow is staged in chunks of at most ch_cols(TZB) x ch_rows(TZB) pixels, so any
// geometry works; typical bricks need one chunk.
//
// What bounds it: at 512^3 x 720, 616 x 480 detector (32-deep bricks) the LDS unit is busy
// for 0.72 of the cycles (a record's read takes it 8 cycles per wavefront) beside 0.92 VALU
// wave-instructions per CU-cycle, of the 1.2 that its mix of operations reaches alone.
// One launch takes 62.7 ms (74.9 ms with a test of every voxel against the brick's top, a
// search for the first and last hit column, an integer clamp made of compares
// and selects, and the ray parameters of a column read again for each of its pixels;
// 65.4 ms before the second row's test was skipped where no voxel of the wavefront has
// one; 64.1 ms before a group of columns with none hit was passed over).  The forms for wider shadows read more records per voxel; split records
// (split_records) halve those reads: 256^3 x 360, 384 x 384 detector 10.5 -> 8.7 -> 8.2 ms.
// EARLY (all but the 32-deep workgroup bricks, whose registers it would spill): 192^3 x 180
// in the wave form 1.97 -> 1.88 ms, 128^3 x 720 1.48 -> 1.38, 256^3 x 90 at 0.7 pixels per
// voxel 0.98 -> 0.88 (both steps).
#pragma once

#pragma clang fp contract(off)

#include <type_traits>

#include "kct_internal.h"
#include "kct_weights.h"

namespace kct {

constexpr int BX = 16, BY = 16, TZ = 16;   // brick; BX * BY = 256 lanes
constexpr int TZ_DEEP = 32;                // deeper bricks for large volumes (more voxels share a lane's setup)
// Rows and columns of the staged chunk by brick depth.  Columns: 32 for the deep bricks of large volumes (whose
// shadows are at most about 28 x 28 pixels at typical magnifications; the
// smaller chunk measured faster there), 48 for the shallow bricks, whose
// volumes tend to have coarse voxels and wide shadows.
__host__ __device__ constexpr int ch_cols(int tzb) { return tzb == TZ_DEEP ? 32 : 48; }
__host__ __device__ constexpr int ch_rows(int tzb) { return tzb == TZ_DEEP ? 36 : 32; }
constexpr int NH = 2;                      // detector columns held in registers at once

// A brick's layers above the volume's top are left out in groups of 4 (a thin volume
// would otherwise cost what a full brick does).  One scalar branch per group; a test
// per voxel costs a scalar condition each, which the compiler keeps in spilled registers.
// Measured (us, no test / groups of 8 / 4 / 2 / 1): 1024^2 x 1 at 0.7 pixels per voxel, 1 view
// 20.3 / 12.8 / 11.6 / 11.7 / 12.1; 1024^2 x 2, 60 views 890 / 424 / 351 / 318 / 319; 1024^2 x 20,
// 8 views 134 / 113 / 102 / 104 / 109; 256^3 x 360 8165 / 8183 / 8119 / 9118 / 9296; 192^3 x 180
// 1606 / 1618 / 1611 / 2096 / 2137; 512^3 x 720 (ms) 64.8 / 64.7 / 64.8 / 65.6 / 67.7.
// Double precision in bricks up to 16 deep: groups of 2, which cost full bricks nothing
// there (groups of 4 / 2 / 1: 1024^2 x 1 at 1.25 pixels per voxel, 8 views 78.6 / 67.3 / 69.2,
// 60 views 561 / 476 / 484; 256^3 x 20 657 / 658 / 684; 32-deep, 128^3 x 60 89.8 / 97.2 / 103).
// Bricks of 32 layers by wavefronts: no test (128^3 x 720, groups of 4 / 16 / no test 1368 / 1371 /
// 1349); volumes that would fill less than five sevenths of them take shallower ones
// (16- / 32-deep: 256^2 x 68, 30 views 113 / 119; double precision, 115 x 261 x 71, 37 views 80 / 71).
template <typename A> __host__ __device__ constexpr bool layer_test(int j, int tzb, bool waves)
{
    if (j == 0 || (tzb == TZ_DEEP && waves)) return false;
    return j % (sizeof(A) == 8 && tzb < TZ_DEEP ? 2 : 4) == 0;
}

struct ColStage {  // per staged detector column: in-plane ray parameters
    float eta_c, inv_a, tcv;  // ColParam's; columns parallel to the eta planes staged as below (PAR_INV)
    float gz;      // d T / d xi with T = (segment fraction) / vz
    float kz;      // ColParam's: d xi / d zeta per unit of a row's factor
};

// Rays parallel to a family of planes are staged as if they crossed them at a
// very steep slope (PAR_INV, in kct_internal.h), with their coordinate on
// that axis moved to the middle of the cell they lie in: every plane is then
// crossed at least half that far from the origin, far outside any xi-interval
// (finite, so the two crossings of a cell never give inf - inf), and the general
// crossing formula gives exactly the parallel-ray intervals of kct_weights.h:
// everything inside the ray's cell, nothing elsewhere.  Staged records and
// columns therefore need no parallel case.

// Per staged pixel: its ray's zeta_offset nzc (from zeta at xi = 0: zeta_centre and
// zeta_inv_slope of its row and column; rows whose rays are parallel to the z-planes
// (qz == 0) staged as above), its d xi / d zeta czr, and L * e in the accumulator precision.
// SPLIT: without czr, which is then the product of the row's staged factor and the
// column's (zeta_inv_slope, the same bits).  A record of 16 bytes takes the LDS 8 cycles
// per wavefront, one of 8 bytes 4 and a row factor 2, for one multiplication and
// one address more.  See split_records.
template <typename A, bool SPLIT> struct PixStage {
    float nzc, czr;
    A le;
    float pad;
};
template <> struct PixStage<double, false> {
    float nzc, czr;
    double le;
};
template <> struct PixStage<float, true> {
    float nzc, le;
};

// Whether bricks tzb voxels deep are staged in split records.  The deepest are chosen
// where a voxel spans less than about a pixel, and are bound by VALU issue (512^3 x 720,
// full / split: 63.7 / 64.3 ms; 400^3 x 60 at 0.7 pixels per voxel 1.83 / 1.93; 128^3 x 720
// 1.39 / 1.43); the others read more records per voxel and the LDS was what bound them
// (192^3 x 180, 256 x 256 detector: 1.89 / 1.63 ms; 192^3 x 120 at 1.6 and 2.2 pixels per
// voxel 2.12 / 1.68 and 4.13 / 3.36; 256^3 x 360 8.64 / 8.21; 64^3 x 90 96 / 85 us).
// In double precision a record is 16 bytes either way.
template <typename A> __host__ __device__ constexpr bool split_records(int tzb)
{
    return std::is_same<A, float>::value && tzb < TZ_DEEP;
}

// 1 / x to within a few ulp (bounds only).
__host__ __device__ __forceinline__ float rcp_approx(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rcpf(x);
#else
    return 1.0f / x;
#endif
}

// Detector coordinates (column, row; fractional pixel indices) of the ray
// through world point (px, py, pz) in view vp.  Used for bounds only.
__host__ __device__ __forceinline__ void project_point(const GeoDev &g, const ViewParam &vp, float px, float py,
                                                       float pz, float &fu, float &fv)
{
    const float dx = px - vp.sx, dy = py - vp.sy;
    const float num = -vp.s * dx + vp.c * dy;
    const float den = -vp.c * dx - vp.s * dy;  // depth along the central ray (> 0)
    const float inv = rcp_approx(den);
    fu = __builtin_fmaf(num * inv, g.ku, g.fu0);
    fv = __builtin_fmaf(pz * inv, g.kv, g.fv0);
}

// Median of x, a and b: x clamped to the interval between a and b.
__host__ __device__ __forceinline__ float med3f(float x, float a, float b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_fmed3f(x, a, b);
#else
    return fmaxf(fminf(x, a), fminf(fmaxf(x, a), b));
#endif
}

// Candidate detector columns [ua, ub] of the voxel column whose in-plane centre
// is (xc, yc): the projective image of its square, bounded around the image of
// the centre (a bound with margin; the weight function decides).
__host__ __device__ __forceinline__ void voxel_columns(const GeoDev &g, const ViewParam &vp, float xc, float yc,
                                                       int &ua, int &ub)
{
    // bounds only: fused multiply-adds round differently from the separate
    // operations by ~1e-7 relative, far inside the 0.01-column margin
    const float dx = xc - vp.sx, dy = yc - vp.sy;
    const float num = __builtin_fmaf(vp.c, dy, -vp.s * dx);
    const float den = __builtin_fmaf(-vp.c, dx, -vp.s * dy);
    const float inv = rcp_approx(den);
    const float inv2 = rcp_approx(den - vp.dd);  // dd: half extent along depth, dn: along e_u
    const float fc = __builtin_fmaf(num * inv, g.ku, g.fu0);
    const float hc = __builtin_fmaf(__builtin_fmaf(vp.dd * fabsf(num), inv, vp.dn) * inv2, g.ku, 0.01f);
    ua = (int)ceilf(fc - hc);
    ub = (int)floorf(fc + hc);
}

// xi-interval [lo, hi] in which the rays of a staged detector column cross the
// voxel column whose xi-cell starts at lo_xi and whose eta-cell is ieta (empty
// when hi <= lo): cell_range of kct_weights.h without its parallel case, which
// the staging removed (PAR_INV).
__host__ __device__ __forceinline__ void column_interval(const ColStage &cs, float lo_xi, int ieta, float heta,
                                                         float &lo, float &hi)
{
    const float mb = (float)ieta - heta;
    const float b0 = cross_at(mb, cs.eta_c, cs.inv_a), b1 = cross_at(mb + 1.0f, cs.eta_c, cs.inv_a);
    lo = fmaxf(lo_xi, fminf(b0, b1));
    hi = fminf(lo_xi + 1.0f, fmaxf(b0, b1));
}

// The staged form of a detector column (view with in-plane domain dom).
__host__ __device__ __forceinline__ ColStage stage_column(const GeoDev &g, int dom, const ColParam &cp)
{
    ColStage cs;
    const bool par = cp.inv_a == 0.0f;
    const float heta = dom == 0 ? g.hy : g.hx;
    cs.eta_c = par ? ((float)parallel_cell(cp.eta_c, heta) - heta) + 0.5f : cp.eta_c;
    cs.inv_a = par ? PAR_INV : cp.inv_a;
    cs.tcv = cp.tcv;
    cs.gz = cp.gp * g.inv_vz;
    cs.kz = cp.kz;
    return cs;
}

// One staged record, read as a whole (one LDS read).
template <typename A, bool SPLIT> __host__ __device__ __forceinline__ PixStage<A, SPLIT> load_pix(const PixStage<A, SPLIT> *p)
{
    return *p;
}
template <> __host__ __device__ __forceinline__ PixStage<float, false> load_pix<float, false>(const PixStage<float, false> *p)
{
    const float4 v = *reinterpret_cast<const float4 *>(p);
    return {v.x, v.y, v.z, v.w};
}
template <> __host__ __device__ __forceinline__ PixStage<float, true> load_pix<float, true>(const PixStage<float, true> *p)
{
    const float2 v = *reinterpret_cast<const float2 *>(p);
    return {v.x, v.y};
}

// One staged record, read where this stands: a volatile access, which the compiler
// does not move down to the record's first use (on the host a plain read).
template <typename A, bool SPLIT> __host__ __device__ __forceinline__ PixStage<A, SPLIT> early_pix(const PixStage<A, SPLIT> *p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (std::is_same<A, float>::value) {
        typedef float record __attribute__((ext_vector_type(SPLIT ? 2 : 3)));
        typedef const volatile __attribute__((address_space(3))) record *lds_record;
        typedef const __attribute__((address_space(3))) PixStage<A, SPLIT> *lds_pix;
        const record v = *(lds_record)(lds_pix)p;
        PixStage<A, SPLIT> r{};
        r.nzc = v.x;
        if constexpr (SPLIT) {
            r.le = v.y;
        } else {
            r.czr = v.y;
            r.le = v.z;
        }
        return r;
    }
#endif
    return *p;
}

// A row's staged factor, read likewise.
__host__ __device__ __forceinline__ float early_row(const float *p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const volatile __attribute__((address_space(3))) float *lds_early;
    typedef const __attribute__((address_space(3))) float *lds_float;
    return *(lds_early)(lds_float)p;
#else
    return *p;
#endif
}

// d xi / d zeta of a staged ray in a row of factor `row` and a column of factor kz.
template <typename A, bool SPLIT>
__host__ __device__ __forceinline__ float pix_slope(const PixStage<A, SPLIT> &p, float row, float kz)
{
    if constexpr (SPLIT) return zeta_inv_slope(row, kz);
    else return p.czr;
}

// The candidate of one record for one voxel with z-planes mb and mb1, over the
// in-plane xi-interval [lo, hi], lo <= hi: a + w * (L e) (w^2 * le when SQ).
// med3(hi, b0, b1) - med3(lo, b0, b1) is the overlap min(hi, max(b0, b1)) -
// max(lo, min(b0, b1)) wherever that is positive (both medians then pick those
// operands) and exactly 0 elsewhere (both medians clamp to the same end of
// [min, max], or hi = lo): a candidate that misses adds 0 * le = 0 (le is finite)
// and leaves the sum as it is.
template <typename A, bool SQ, bool SPLIT>
__host__ __device__ __forceinline__ A add_pix(const PixStage<A, SPLIT> &p, float czr, float lo, float hi, float mb, float mb1, A a)
{
    const float b0 = zeta_cross(mb, p.nzc, czr), b1 = zeta_cross(mb1, p.nzc, czr);
    const float w = med3f(hi, b0, b1) - med3f(lo, b0, b1);
    return fma_acc(SQ ? w * w : w, p.le, a);
}

// The candidates of one detector row for one voxel: the rays of the row in the
// nh (<= NH) staged hit columns starting at prow, whose in-plane xi-intervals
// are [lo[h], hi[h]] with lo[h] <= hi[h], against the voxel's z-planes mb and
// mb1.  Returns a + sum of w * (L e) (w^2 * le when SQ).  All NH records are
// read before the first is used; the staging buffer holds a spare record past
// its last, so prow + NH - 1 is always inside it.
template <typename A, bool SQ, int NH, bool SPLIT>
__host__ __device__ __forceinline__ A add_row(const PixStage<A, SPLIT> *prow, float row, int nh, const float (&kz)[NH],
                                              const float (&lo)[NH], const float (&hi)[NH], float mb, float mb1, A a)
{
    PixStage<A, SPLIT> p[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) p[h] = load_pix(prow + h);
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        if (h == 0 || h < nh) a = add_pix<A, SQ>(p[h], pix_slope(p[h], row, kz[h]), lo[h], hi[h], mb, mb1, a);
    }
    return a;
}

// The staged record of the pixel with column parameters cp, row parameters rp
// and value ev (parallel rows as above).  SQ: L^2 in the place of L * ev.
template <typename A, bool SQ, bool SPLIT>
__host__ __device__ __forceinline__ PixStage<A, SPLIT> stage_pixel(const ColParam &cp, const RowParam &rp, A ev)
{
    PixStage<A, SPLIT> ps;
    const float czr = zeta_inv_slope(rp.s_inv, cp.kz);
    if constexpr (!SPLIT) ps.czr = czr;
    ps.nzc = zeta_offset(zeta_centre(rp.qz, cp.tcv, -rp.s_off), czr);
    const A L = (A)ray_length_per_xi(cp.lxy2, rp.qz, cp.gp);
    ps.le = SQ ? L * L : L * ev;
    return ps;
}

// A record of weight 0 for any voxel, made where it is stored (an empty asm keeps
// the compiler from hoisting it out of the view loop and spilling it).
template <typename A, bool SPLIT> __host__ __device__ __forceinline__ PixStage<A, SPLIT> zero_pixel()
{
    float zero = 0.0f;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(zero));
#endif
    PixStage<A, SPLIT> z{};
    z.nzc = zero;
    if constexpr (!SPLIT) z.czr = zero;
    z.le = (A)zero;
    return z;
}

// pg + r * stride for a pointer pg into the LDS staging buffer, stride records per
// staged row: CHC, or the run-time value (equal in every lane) where CHC is 0.  On
// the GPU one instruction on the 32-bit LDS address: a shift-and-add when a
// row of records spans a constant power of two bytes, else a 24-bit
// multiply-and-add (row and row length are far below 2^23).
template <int CHC, typename A, bool SPLIT>
__host__ __device__ __forceinline__ const PixStage<A, SPLIT> *row_record(const PixStage<A, SPLIT> *pg, int r, int stride)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr unsigned row_bytes = CHC * sizeof(PixStage<A, SPLIT>);
    if constexpr ((row_bytes & (row_bytes - 1)) == 0) {
        typedef const __attribute__((address_space(3))) PixStage<A, SPLIT> *lds_rec;
        const unsigned base = (unsigned)(size_t)(lds_rec)pg;
        unsigned addr;
        if constexpr (CHC != 0)
            asm("v_lshl_add_u32 %0, %1, %3, %2" : "=v"(addr) : "v"(r), "v"(base), "i"(__builtin_ctz(row_bytes)));
        else
            asm("v_mad_i32_i24 %0, %1, %3, %2" : "=v"(addr) : "v"(r), "v"(base), "s"(stride * (int)sizeof(PixStage<A, SPLIT>)));
        return (const PixStage<A, SPLIT> *)(lds_rec)(size_t)addr;
    }
#endif
    return pg + r * (CHC != 0 ? CHC : stride);
}

// rg + r for a pointer rg into the LDS: one shift-and-add of the 32-bit address on the GPU.
__host__ __device__ __forceinline__ const float *row_factor(const float *rg, int r)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const __attribute__((address_space(3))) float *lds_float;
    const unsigned base = (unsigned)(size_t)(lds_float)rg;
    unsigned addr;
    asm("v_lshl_add_u32 %0, %1, 2, %2" : "=v"(addr) : "v"(r), "s"(base));
    return (const float *)(lds_float)(size_t)addr;
#else
    return rg + r;
#endif
}

// Whether c holds in any lane of the wavefront: a scalar value on the GPU.
__host__ __device__ __forceinline__ bool any_lane(bool c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ballot_w64(c) != 0;
#else
    return c;
#endif
}

// v clamped to [-1, hi] (hi >= -1 equal in every lane): one instruction on the GPU.
__host__ __device__ __forceinline__ int clamp_row(int v, int hi)
{
#if defined(__HIP_DEVICE_COMPILE__)
    int r;
    asm("v_med3_i32 %0, %1, -1, %2" : "=v"(r) : "v"(v), "s"(hi));
    return r;
#else
    return v < -1 ? -1 : (v > hi ? hi : v);
#endif
}

// The voxels of one lane for one group of hit columns: voxel j has the planes
// mbz0 + j and mbz0 + j + 1 and, counted from the first staged row, the candidate
// rows va + 1 .. vb + 1 with va = floor(l0 + j sl) and vb = floor(h0 + (j + 1) sh).
// `layers` of the TZN voxels lie in the volume (the same in every lane); those above are
// left out from the next group on (layer_test; the others' sums are never stored).
// The first candidate row is evaluated for every voxel, without a
// branch: va is clamped to [-1, nrow - 1], so row va + 1 is a staged row or the zero
// row staged after them, and a row that is not a candidate has weight exactly
// 0 (the weights are exact).  Further rows, up to the last staged one, follow in a
// loop.  pg + va * stride is the record of row va + 1 in the group's first column.
template <typename A, bool SQ, int CHC, int NH, bool EARLY, int TZN, bool SPLIT>
__host__ __device__ __forceinline__ void voxel_rows(const PixStage<A, SPLIT> *pg, const float *rg, int stride, int nh,
                                                    const float (&kz)[NH], const float (&lo)[NH],
                                                    const float (&hi)[NH], float mbz0, float l0, float sl,
                                                    float h0, float sh, int nrow, int layers, A (&acc)[TZN])
{
    // The per-voxel plane values do not depend on the column group; computed
    // here they stay short-lived (hoisted out of the group loop, all TZ of them
    // would stay live through it).  The empty asm keeps the compiler from
    // hoisting them.
    float mbb = mbz0;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(mbb));
#endif
    float mb = mbb;  // lower plane of voxel j (exact: an integer or half-integer)
    // Whether some voxel of some lane has a second candidate row.  vhi - vlo is linear in j
    // and negative at both ends where no voxel has (the margin is far above its rounding).
    const float len0 = (h0 + sh) - l0, len1 = len0 + (float)(TZN - 1) * (sh - sl);
    const bool more = any_lane(fmaxf(len0, len1) > -1.0e-3f);
    // EARLY: the next voxel's first record is read before this voxel's arithmetic (its
    // latency is then covered; it takes four more registers)
    int va = clamp_row((int)floorf(l0), nrow - 1);
    const PixStage<A, SPLIT> *prow = row_record<CHC>(pg, va, stride);
    PixStage<A, SPLIT> rec{};
    float row = 0.0f;
    if constexpr (EARLY) {
        if constexpr (SPLIT) row = early_row(row_factor(rg, va));
        rec = early_pix(prow);
    }
#pragma unroll
    for (int j = 0; j < TZN; ++j) {
        if (layer_test<A>(j, TZN, CHC == 0) && j >= layers) break;
        const float mb1 = mb + 1.0f;
        // candidate rows va + 1 .. vb + 1: floor(lo) + 1 is ceil(lo) except at an
        // integer lo, whose row lies 0.01 below the true bound and is rightly left out
        int va_next = va;
        const PixStage<A, SPLIT> *prow_next = prow;
        PixStage<A, SPLIT> rec_next = rec;
        float row_next = row;
        if constexpr (EARLY) {
            if (j + 1 < TZN) {
                va_next = clamp_row((int)floorf(__builtin_fmaf((float)(j + 1), sl, l0)), nrow - 1);
                prow_next = row_record<CHC>(pg, va_next, stride);
                if constexpr (SPLIT) row_next = early_row(row_factor(rg, va_next));
                rec_next = early_pix(prow_next);
            }
            acc[j] = add_pix<A, SQ>(rec, pix_slope(rec, row, kz[0]), lo[0], hi[0], mb, mb1, acc[j]);
#pragma unroll
            for (int h = 1; h < NH; ++h) {
                if (h < nh) {
                    const PixStage<A, SPLIT> p = load_pix(prow + h);
                    acc[j] = add_pix<A, SQ>(p, pix_slope(p, row, kz[h]), lo[h], hi[h], mb, mb1, acc[j]);
                }
            }
        } else {
            if (j > 0) {
                va = clamp_row((int)floorf(__builtin_fmaf((float)j, sl, l0)), nrow - 1);
                prow = row_record<CHC>(pg, va, stride);
            }
            if constexpr (SPLIT) row = *row_factor(rg, va);
            acc[j] = add_row<A, SQ, NH>(prow, row, nh, kz, lo, hi, mb, mb1, acc[j]);
        }
        if (more) {
            int vb = (int)floorf(__builtin_fmaf((float)(j + 1), sh, h0));
            vb = vb > nrow - 2 ? nrow - 2 : vb;
            A a = acc[j];
            const float *prf = rg;
            float further = 0.0f;
            if constexpr (SPLIT) prf = row_factor(rg, va);
            for (int v = va; v < vb; ++v) {
                prow += CHC != 0 ? CHC : stride;
                if constexpr (SPLIT) further = *++prf;
                a = add_row<A, SQ, NH>(prow, further, nh, kz, lo, hi, mb, mb1, a);
            }
            acc[j] = a;
        }
        if constexpr (EARLY) {
            va = va_next;
            prow = prow_next;
            rec = rec_next;
            row = row_next;
        }
        mb = mb1;
    }
}

// One lane's share of one staged chunk of one view: add w_ij * (L_i e_i) to the
// accumulators of its voxels (ix, iy, iz0 + j), j < layers <= TZN, for every staged ray
// i = (column cu0 + c, row cv0 + r); s_pix[r * stride + c] describes ray i (stride:
// CHC, or the argument where CHC is 0), and row nrow of s_pix holds zero records
// (weight 0 for any voxel).  NH columns are taken at once.
// SQ: accumulate w_ij^2 * le instead of w_ij * le (with le = L^2 this sums the
// squared weights, the diagonal of A^T A).
template <typename A, bool SQ, int CHC, int NH, bool EARLY, int TZN, bool SPLIT>
__host__ __device__ __forceinline__ void gather_chunk(const GeoDev &g, const ViewParam &vp, int ix, int iy, int iz0,
                                                      const PixStage<A, SPLIT> *s_pix, const ColStage *s_col,
                                                      const float *s_row, int cu0,
                                                      int ncol, int cv0, int nrow, int layers, A (&acc)[TZN], int stride = CHC)
{
    int ixi, ieta;
    float hxi, heta;
    if (vp.dom == 0) { ixi = ix; ieta = iy; hxi = g.hx; heta = g.hy; }
    else { ixi = iy; ieta = ix; hxi = g.hy; heta = g.hx; }
    const float lo_xi = (float)ixi - hxi;
    int ua, ub;
    voxel_columns(g, vp, g.x0 + ((float)ix + 0.5f) * g.vx, g.y0 + ((float)iy + 0.5f) * g.vy, ua, ub);
    ua = ua < cu0 ? cu0 : ua;
    ub = ub > cu0 + ncol - 1 ? cu0 + ncol - 1 : ub;
    const float mbz0 = (float)iz0 - g.hz;  // lower plane of the first voxel (index frame)
    const float zz0 = mbz0 + g.zc;         // the same plane as a height above the source plane
    // row coordinates from the first staged row; the upper bound one row lower, as
    // voxel_rows takes it
    const float fv = g.fv0 - (float)cv0, vofs_lo = fv - 0.01f, vofs_hi = fv - 0.99f;
    // The bound [ua, ub] is met by nearly every column in it (its margin is 0.01
    // column, and it takes the square's extents across and along the central ray
    // as independent): one column more at either end where a voxel spans fewer than
    // about five pixels.  Those that are missed are left out, so that a value that is not
    // finite reaches no voxel column that its detector column misses: at the far end
    // by nh, at the near end by a test here, or, for the deep bricks, where it is
    // cheaper, by moving the group on by one.  Measured (us, ends left in / test / moved on): 512^3 x
    // 720 (ms) 64.3 / 63.8 / 63.1; 256^3 x 360 8085 / 8050 / 8145; 96^3 x 186 592 / 585 / 605; 64^3 x 90
    // 76.8 / 77.8 / 78.7; 192^3 x 180 1606 / 1622 / 1621.  (All columns tested for the first and the
    // last hit one cost 2 to 4 % more.)
    constexpr bool MOVE = TZN == TZ_DEEP;
    static_assert(!MOVE || NH == 2, "a hit group of two has at most one column to pass over");
    if constexpr (!MOVE) {
        float lo, hi;
        column_interval(s_col[ua < cu0 + ncol ? ua - cu0 : 0], lo_xi, ieta, heta, lo, hi);
        ua += hi > lo ? 0 : 1;
    }
    for (int c0 = ua; c0 <= ub; c0 += NH) {
        // xi-intervals of up to NH columns, and the range of T = tcv + xi gz over
        // those that are hit (a ray of height qz is at height qz T above the source plane)
        const int in = ub - c0 + 1 < NH ? ub - c0 + 1 : NH;
        int nh = 1, first = 0;  // columns taken, and those passed over before them
        float lo[NH], hi[NH], kz[NH];
        float tmin = INFINITY, tmax = 0.0f;
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int c = h < in ? c0 + h : c0;
            const ColStage cs = s_col[c - cu0];
            kz[h] = cs.kz;
            column_interval(cs, lo_xi, ieta, heta, lo[h], hi[h]);
            if (h < in && hi[h] > lo[h]) {
                nh = h + 1;
                const float T1 = __builtin_fmaf(lo[h], cs.gz, cs.tcv), T2 = __builtin_fmaf(hi[h], cs.gz, cs.tcv);
                tmin = fminf(tmin, fminf(T1, T2));
                tmax = fmaxf(tmax, fmaxf(T1, T2));
            }
        }
        if (!(tmax > 0.0f)) continue;  // no column of this group is hit
        if constexpr (MOVE) {
            first = hi[0] > lo[0] ? 0 : 1;
            nh -= first;
#pragma unroll
            for (int h = 0; h + 1 < NH; ++h) {
                lo[h] = first ? lo[h + 1] : lo[h];
                hi[h] = first ? hi[h + 1] : hi[h];
                kz[h] = first ? kz[h + 1] : kz[h];
            }
        }
#pragma unroll
        for (int h = MOVE ? 1 : 0; h < NH; ++h) hi[h] = fmaxf(hi[h], lo[h]);  // an empty interval becomes [lo, lo]: its weights are 0 (add_row)
        // Rows: inside these columns a ray of row height qz meets the z-cell with
        // planes at heights [zz, zz + 1] only if qz lies in [zz, zz + 1] / [Tmin, Tmax].
        // In row units a plane at height z bounds the rows from below by
        // f_lo(z) = min(z ra, z rb) and from above by f_hi(z) = max(z ra, z rb).
        // f_lo is concave and f_hi convex in z, so over the brick's planes the
        // chords between its lowest and highest plane bound them from the safe
        // side (exactly equal to them unless the brick straddles the source
        // plane z = 0): plane p gives lo_p = l0 + p sl and hi_p = h0 + p sh, one
        // fused multiply-add each.  Their rounding (~1e-5 row) is far inside the
        // 0.01-row margins.
        const float ra = __builtin_amdgcn_rcpf(tmax) * g.inv_dv, rb = __builtin_amdgcn_rcpf(tmin) * g.inv_dv;
        const float za = zz0, zb = zz0 + (float)TZN;  // lowest and highest plane of the brick
        const float a1 = za * ra, a2 = za * rb, b1 = zb * ra, b2 = zb * rb;
        const float sl = (fminf(b1, b2) - fminf(a1, a2)) * (1.0f / TZN);
        const float sh = (fmaxf(b1, b2) - fmaxf(a1, a2)) * (1.0f / TZN);
        const float l0 = fminf(a1, a2) + vofs_lo, h0 = fmaxf(a1, a2) + vofs_hi;
        const PixStage<A, SPLIT> *pg = s_pix + ((c0 + first - cu0) + (CHC != 0 ? CHC : stride));  // row va + 1 at pg + va * stride
        voxel_rows<A, SQ, CHC, NH, EARLY>(pg, s_row + 1, stride, nh, kz, lo, hi, mbz0, l0, sl, h0, sh, nrow, layers, acc);
    }
}

}  // namespace kct
