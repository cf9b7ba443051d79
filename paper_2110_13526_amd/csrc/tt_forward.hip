// tt_forward.hip -- the TT footprint projector's forward, p = A x (kct_tt.h), with
// single-precision accumulation.
//
// A workgroup holds TTF_COLS neighbouring detector columns and 64 R detector rows of one
// view; its four wavefronts take every fourth group of slabs of the view's dominant
// axis, and their sums are added at the end.  For the voxel columns of the wedge that
// the detector columns see in its slabs, a wavefront
//   1. computes the transaxial footprints, one voxel column per lane, and lists
//      in LDS those that meet a detector column (z-column, depths, row scales, F_u of
//      each of the detector columns),
//   2. takes the list entry by entry (the same in every lane): each lane sums
//      F_v x over the z-cells whose axial footprint meets its row, once for all
//      detector columns, and adds it with each column's F_u.
// Bounded by VALU issue.  With one detector column per wavefront, every lane computing
// every transaxial footprint and every row's axial sum once per detector column, 128^3 x
// 180 views, 154 x 120 detector took 4.47 ms; this form 1.33 ms (each step: lists and shared axial
// sums 1.93, planes shared by neighbouring cells 1.69, by neighbouring rows 1.44).
// 512^3 x 720, 616 x 480: 879 -> 279 ms.
#include <type_traits>

#include "kct_epilogue.h"
#include "kct_internal.h"
#include "kct_ray.h"
#include "kct_tt.h"
#include "kct_weights.h"

namespace kct {

// Detector columns of a workgroup: more share each list and axial sum, fewer keep more
// wavefronts in flight.  4 / 8 / 16 (us; cube of n voxels, q detector pixels per voxel): n 96,
// q 4, 20 views 421 / 361 / 541; n 192, q 2.2, 30 views 1891 / 1715 / 2301, q 1.25 1101 / 1092 / 1625, q 0.7, 60
// views 1997 / 2229 / 3222; n 128, q 0.7, 60 views 584 / 868 / 1262; n 32, q 1.25, 30 views 42 / 68 / 138.
constexpr int TTF_COLS = 8;
constexpr int TTF_WAVES = 4;
// Lanes per slab when the footprints are listed.  8 / 16 / 32: n 96, q 4 345 / 361 / 410; n 192,
// q 2.2 1642 / 1715 / 1877, q 0.7 2238 / 2229 / 2280; n 128, q 0.83, 180 views 1366 / 1338 / 1384.
constexpr int TTF_SLOTS = 16;
constexpr int TTF_SLABS = 64 / TTF_SLOTS;

struct TTFEntry {               // one voxel column that the detector columns see
    int column;                 // iy * nx + ix
    float dmin, dmax;           // least and greatest depth of its corners [mm]
    int mask;                   // detector columns with F_u > 0
    float ka, kb;               // row scales at dmin and dmax
    float pad[2];
    float fu[TTF_COLS];
};

struct TTFGrid {
    int ncg, nbands, nviews, rows;
    int64_t nblocks;
};

// (two neighbouring rows per lane; one where the detector has no more than 64)
__host__ __device__ __forceinline__ TTFGrid ttf_grid(const GeoDev &g)
{
    TTFGrid f;
    f.rows = g.nv > 64 ? 2 : 1;
    f.ncg = (g.nu + TTF_COLS - 1) / TTF_COLS;
    f.nbands = (g.nv + 64 * f.rows - 1) / (64 * f.rows);
    f.nviews = g.nviews;
    f.nblocks = (int64_t)f.ncg * f.nbands * f.nviews;
    return f;
}

int64_t tt_forward_num_blocks(const GeoDev &g) { return ttf_grid(g).nblocks; }

__device__ __forceinline__ void ttf_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename TV, typename TP, int EPI, int R, bool OVERLAP, bool ZFAST>
__global__ __launch_bounds__(256, 5) void k_forward_tt(GeoDev g, const TV *__restrict__ vol, const TV *__restrict__ vol_z,
                                                       TP *__restrict__ out, const TP *__restrict__ aux,
                                                       const Scalars *__restrict__ sc, double *__restrict__ partials,
                                                       const int *__restrict__ skip)
{
    constexpr int SUMS = TTF_WAVES * TTF_COLS * R * 64;  // every wavefront's sums, after the lists
    constexpr size_t LISTS = sizeof(TTFEntry) * 64 * TTF_WAVES;
    __shared__ __align__(16) char lds[LISTS > SUMS * sizeof(float) ? LISTS : SUMS * sizeof(float)];
    __shared__ double red[TTF_WAVES];
    if (skip && *skip) return;
    const int tid = (int)__builtin_amdgcn_workitem_id_x();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    TTFEntry *list = reinterpret_cast<TTFEntry *>(lds) + wave * 64;
    // column group fastest, then view, then band; within 64 consecutive workgroups
    // each XCD gets 8 neighbouring groups
    const TTFGrid fg = ttf_grid(g);
    const int64_t w = __builtin_amdgcn_workgroup_id_x();
    const int64_t full = fg.nblocks & ~(int64_t)63;
    const int64_t at = w < full ? (w & ~(int64_t)63) + (w % 8) * 8 + (w / 8) % 8 : w;
    const int iu0 = (int)(at % fg.ncg) * TTF_COLS;
    const int64_t rest = at / fg.ncg;
    const int k = (int)(rest % fg.nviews), iv0 = (int)(rest / fg.nviews) * 64 * R;
    const int ncols = g.nu - iu0 < TTF_COLS ? g.nu - iu0 : TTF_COLS;
    const ViewParam vp = g.views[k];
    const bool dom0 = vp.dom == 0;
    const int nxi = dom0 ? g.nx : g.ny, neta = dom0 ? g.ny : g.nx;
    const float hxi = dom0 ? g.hx : g.hy, heta = dom0 ? g.hy : g.hx;
    // lines through the source and the outer edges of the detector columns: eta = a0 + a1 xi, b0 + b1 xi
    float a0, a1, b0, b1;
    tt_edge_line(g, vp, (float)iu0 - 0.5f, a0, a1);
    tt_edge_line(g, vp, (float)(iu0 + ncols) - 0.5f, b0, b1);
    // the lane's rows iv0 + lane R + r: the first one's pixel, and the ends of all of
    // them on the detector per depth, in z-cells
    const float um0 = (float)(iv0 + lane * R) - 0.5f;
    const float to_cells = 1.0f / g.sdd * g.inv_vz;
    const float zcell0 = g.z0 * g.inv_vz;
    const float vlo = ((um0 - g.cv) * g.dv + g.off_v) * to_cells;
    const float vhi = ((um0 + (float)R - g.cv) * g.dv + g.off_v) * to_cells;
    const float roff = tt_row_offset(g);

    float acc[TTF_COLS][R];
#pragma unroll
    for (int c = 0; c < TTF_COLS; ++c)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[c][r] = 0.0f;

    // F_v x summed over the z-cells of one voxel column that meet the lane's pixels, for
    // each of them: neighbouring rows share the planes between (and the loads)
    auto axial_sums = [&](int column, float dmin, float dmax, float ka, float kb, float (&sum)[R]) {
#pragma unroll
        for (int r = 0; r < R; ++r) sum[r] = 0.0f;
        // the z-cells meeting the pixels' range at either depth, widened by 0.01 cell
        // against the rounding differences to the ramps
        const float l0 = vlo * dmin, l1 = vlo * dmax, h0 = vhi * dmin, h1 = vhi * dmax;
        int za = (int)floorf(fminf(l0, l1) - zcell0 - 0.01f), zb = (int)floorf(fmaxf(h0, h1) - zcell0 + 0.01f);
        za = za < 0 ? 0 : za;
        zb = zb > g.nz - 1 ? g.nz - 1 : zb;
        if (za > zb) return;
        float plane = (float)za;  // (exact: a volume side is at most 2^20)
        TTRamp p0 = tt_plane_ramp(g, plane, ka, kb, roff);
        float i0[R];
#pragma unroll
        for (int r = 0; r < R; ++r) i0[r] = OVERLAP ? 0.0f : tt_ramp_mean(p0, um0 + (float)r, um0 + (float)(r + 1));
        for (int iz = za; iz <= zb; ++iz) {
            TV x;
            if constexpr (ZFAST) x = ZCol<TV, 1>(vol_z + (size_t)column * g.nz, g.nz, 1).raw(iz * ZCol<TV, 1>::UNIT);
            else x = vol[(size_t)iz * g.nx * g.ny + column];
            plane += 1.0f;
            const TTRamp p1 = tt_plane_ramp(g, plane, ka, kb, roff);
            float fv[R];
            if constexpr (OVERLAP) {
                TTRamp a, b;
                tt_layer_ramps<OVERLAP>(p0, p1, a, b);
#pragma unroll
                for (int r = 0; r < R; ++r) fv[r] = tt_trap_mean(a, b, um0 + (float)r, um0 + (float)(r + 1));
                p0 = p1;
            } else {  // tt_trap_mean with the plane's mean carried from the layer below
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float i1 = tt_ramp_mean(p1, um0 + (float)r, um0 + (float)(r + 1));
                    fv[r] = fmaxf(i0[r] - i1, 0.0f);
                    i0[r] = i1;
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (fv[r] > 0.0f) sum[r] = __builtin_fmaf(fv[r], to_f32(x), sum[r]);
        }
    };

    for (int m0 = wave * TTF_SLABS; m0 < nxi; m0 += TTF_WAVES * TTF_SLABS) {
        // the eta-cells of this lane's slab inside the wedge, widened by 0.01 cell against
        // the rounding differences to tt_transaxial's breakpoints
        const int m = m0 + lane / TTF_SLOTS;
        const float xl = (float)m - hxi, xh = xl + 1.0f;
        const float ea = a0 + a1 * xl, eb = a0 + a1 * xh, ec = b0 + b1 * xl, ed = b0 + b1 * xh;
        int e_lo = (int)floorf(fminf(fminf(ea, eb), fminf(ec, ed)) + heta - 0.01f);
        int e_hi = (int)floorf(fmaxf(fmaxf(ea, eb), fmaxf(ec, ed)) + heta + 0.01f);
        e_lo = e_lo < 0 ? 0 : e_lo;
        e_hi = m >= nxi ? -1 : (e_hi > neta - 1 ? neta - 1 : e_hi);
        for (int e = e_lo + lane % TTF_SLOTS; __builtin_amdgcn_ballot_w64(e <= e_hi) != 0; e += TTF_SLOTS) {
            TTFEntry en;
            en.mask = 0;
            if (e <= e_hi) {
                const int ix = dom0 ? m : e, iy = dom0 ? e : m;
                TTTrap tu;
                float rdmin, rdmax;
                tt_transaxial(g, vp, ix, iy, tu, en.dmin, en.dmax, rdmin, rdmax);
                en.column = iy * g.nx + ix;
                tt_row_scales(g, rdmin, rdmax, en.ka, en.kb);
                const TTRamp r0 = tt_ramp(tu.t[0], tu.t[1]), r1 = tt_ramp(tu.t[2], tu.t[3]);
#pragma unroll
                for (int c = 0; c < TTF_COLS; ++c) {
                    const float ul = (float)(iu0 + c) - 0.5f;
                    const float fu = c < ncols ? tt_trap_mean(r0, r1, ul, ul + 1.0f) : 0.0f;
                    en.fu[c] = fu;
                    en.mask |= fu > 0.0f ? 1 << c : 0;
                }
            }
            const uint64_t kept = __builtin_amdgcn_ballot_w64(en.mask != 0);
            if (en.mask != 0) {
                const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(kept >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)kept, 0));
                list[below] = en;
            }
            ttf_lds_order();
            const int n = __builtin_popcountll(kept);
            for (int i = 0; i < n; ++i) {
                const TTFEntry &q = list[i];
                const int column = __builtin_amdgcn_readfirstlane(q.column);
                const int mask = __builtin_amdgcn_readfirstlane(q.mask);
                float s[R];
                axial_sums(column, q.dmin, q.dmax, q.ka, q.kb, s);
#pragma unroll
                for (int c = 0; c < TTF_COLS; ++c) {
                    if (mask & (1 << c)) {
                        const float fu = q.fu[c];
#pragma unroll
                        for (int r = 0; r < R; ++r) acc[c][r] = __builtin_fmaf(fu, s[r], acc[c][r]);
                    }
                }
            }
            ttf_lds_order();
        }
    }

    // the four wavefronts' sums, then the outputs, neighbouring columns in neighbouring threads
    __syncthreads();
    float *sums = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int c = 0; c < TTF_COLS; ++c)
#pragma unroll
        for (int r = 0; r < R; ++r) sums[((wave * TTF_COLS + c) * R + r) * 64 + lane] = acc[c][r];
    __syncthreads();
    double sq = 0.0;
    for (int i = tid; i < TTF_COLS * R * 64; i += 256) {
        const int c = i % TTF_COLS, row = i / TTF_COLS;
        const int iu = iu0 + c, iv = iv0 + row;
        if (c >= ncols || iv >= g.nv) continue;
        float v[TTF_WAVES];
#pragma unroll
        for (int q = 0; q < TTF_WAVES; ++q) v[q] = sums[((q * TTF_COLS + c) * R + row % R) * 64 + row / R];
        const ColParam cp = g.cols[(size_t)k * g.nu + iu];
        const RowParam rp = g.rows[iv];
        const float amp = tt_amplitude(ray_length_per_xi(cp.lxy2, rp.qz, cp.gp), cp.inv_a, zeta_inv_slope(rp.inv_qz, cp.kz));
        const size_t ray = ((size_t)k * g.nv + iv) * g.nu + iu;
        sq += fwd_store<TP, EPI, float>(out, aux, sc, ray, amp * ((v[0] + v[1]) + (v[2] + v[3])));
    }
    if (EPI != FWD_PLAIN) {
        for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
        if (lane == 0) red[wave] = sq;
        __syncthreads();
        if (tid == 0) partials[w] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

template <typename TV, typename TP, int EPI, bool ZFAST>
static hipError_t launch_ftt(const GeoDev &g, const TV *vol, const TV *vol_z, TP *out, const TP *aux, const Scalars *sc,
                             double *partials, const int *skip, hipStream_t st)
{
    const TTFGrid f = ttf_grid(g);
    const dim3 grid((unsigned)f.nblocks), block(64 * TTF_WAVES);
#define KCT_TTF_LAUNCH(R, OVERLAP)                                                                                     \
    hipLaunchKernelGGL((k_forward_tt<TV, TP, EPI, R, OVERLAP, ZFAST>), grid, block, 0, st, g, vol, vol_z, out, aux, sc, \
                       partials, skip)
    if (g.tt_overlap) {
        if (f.rows == 1) KCT_TTF_LAUNCH(1, true);
        else KCT_TTF_LAUNCH(2, true);
    } else {
        if (f.rows == 1) KCT_TTF_LAUNCH(1, false);
        else KCT_TTF_LAUNCH(2, false);
    }
#undef KCT_TTF_LAUNCH
    return hipGetLastError();
}

// The forms that are called: as for the Siddon pair (launch_forward_rows).
template <typename TV, typename TP>
hipError_t launch_forward_tt(const GeoDev &g, const TV *vol, const TV *vol_z, TP *out, const TP *aux, int epi,
                             const Scalars *sc, double *partials, const int *skip, hipStream_t st)
{
    if constexpr (std::is_same<TV, double>::value) {
        return launch_forward_tt_f64(g, vol, vol_z, out, epi, skip, st);
    } else {
        if constexpr (std::is_same<TV, TP>::value) {
            if (epi == FWD_PLAIN)
                return vol_z ? launch_ftt<TV, TP, FWD_PLAIN, true>(g, vol, vol_z, out, aux, sc, partials, skip, st)
                             : launch_ftt<TV, TP, FWD_PLAIN, false>(g, vol, vol_z, out, aux, sc, partials, skip, st);
            if (epi == FWD_NORM && vol_z) return launch_ftt<TV, TP, FWD_NORM, true>(g, vol, vol_z, out, aux, sc, partials, skip, st);
            if (epi == FWD_LSQR && vol_z) return launch_ftt<TV, TP, FWD_LSQR, true>(g, vol, vol_z, out, aux, sc, partials, skip, st);
        }
        if constexpr (std::is_same<TV, float>::value) {
            if (epi == FWD_BMINUS)
                return vol_z ? launch_ftt<TV, TP, FWD_BMINUS, true>(g, vol, vol_z, out, aux, sc, partials, skip, st)
                             : launch_ftt<TV, TP, FWD_BMINUS, false>(g, vol, vol_z, out, aux, sc, partials, skip, st);
        }
        return hipErrorInvalidValue;
    }
}

#define KCT_TTF(TV, TP)                                                                                         \
    template hipError_t launch_forward_tt<TV, TP>(const GeoDev &, const TV *, const TV *, TP *, const TP *, int, \
                                                  const Scalars *, double *, const int *, hipStream_t);
KCT_TTF(float, float)
KCT_TTF(bf16, bf16)
KCT_TTF(_Float16, _Float16)
KCT_TTF(float, bf16)
KCT_TTF(float, _Float16)
KCT_TTF(double, double)

}  // namespace kct
