// kct_forward.h -- the forward cone-beam projector for gfx950.
//
//   forward  p = A x    (Section 2, Eq. 1): ray-driven.  One lane per ray; the
//            lanes of a wavefront hold neighbouring detector rows of one
//            column (R rows per lane).  Their rays share the in-plane part of the walk (identical
//            work in every lane, no divergence), differ only in z, and read a
//            copy of the volume stored z-fastest, so one gather instruction of
//            the wavefront touches a few neighbouring cache lines.  Each lane
//            accumulates w_ij * x_j in single precision (kct_ray.h).
//
// What bounds it: VALU issue for volumes whose z-columns come from the caches (256^3 x 360,
// 384 x 384 detector: 1.16 wave-instructions per CU-cycle), the texture addresser for
// larger ones (512^3 x 720: busy 88 % of the cycles, 0.73 wave-instructions per CU-cycle).
// One piece of a wavefront's walk takes about 69 VALU instructions with four rows (92
// when the crossed cell's step and its read were masked separately and the in-plane step
// was selected instead of branched around).  Measured with the rows-per-lane rule and the
// workgroup order below: 512^3 x 720 59.3 -> 48.5 ms (FP32), 50.5 -> 47.5 (BF16); 256^3 x 360
// 8.64 -> 4.63; 192^3 x 180, 256 x 256 1.43 -> 0.87; 128^3 x 720, 154 x 120 1.50 -> 0.89;
// 64^3 x 90, 96 x 96 131 -> 68 us.
//
// The kernel can fuse a double-precision partial sum of the squares of its
// outputs (|p|^2 of Algorithm 1) and the LSQR bidiagonalisation update.  The
// rows per lane are a template parameter; forward_r1.hip to forward_r4.hip hold
// one instantiation each, projector.hip chooses among them.
#pragma once

#include <type_traits>

#include "kct_epilogue.h"
#include "kct_internal.h"
#include "kct_ray.h"
#include "kct_weights.h"

namespace kct {

constexpr int FWD_COLS = 4;    // detector columns per workgroup (one per wavefront)
constexpr unsigned FWD_XCDS = 8;
constexpr int FWD_PARTS = 4;   // shares of a divided walk

// Sum of v over the first 256 threads of the workgroup, in a fixed order.
// Result is valid in thread 0.
__device__ __forceinline__ double fwd_block_sum(double v)
{
    __shared__ double red[4];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int w = __builtin_amdgcn_workitem_id_x() >> 6;
    if ((__builtin_amdgcn_workitem_id_x() & 63) == 0 && w < 4) red[w] = v;
    __syncthreads();
    double r = 0.0;
    if (__builtin_amdgcn_workitem_id_x() == 0) r = (red[0] + red[1]) + (red[2] + red[3]);
    return r;
}

struct FwdGrid {
    int ncg, nbands, nviews;
    int64_t nblocks;
};

__host__ __device__ __forceinline__ FwdGrid fwd_grid(const GeoDev &g, int rows_per_lane)
{
    FwdGrid f;
    const int rows = 64 * rows_per_lane;  // detector rows per wavefront
    f.ncg = (g.nu + FWD_COLS - 1) / FWD_COLS;
    f.nbands = (g.nv + rows - 1) / rows;
    f.nviews = g.nviews;
    f.nblocks = (int64_t)f.ncg * f.nbands * f.nviews;
    return f;
}

// Workgroup order.  Neighbouring views pass through nearly the same voxels, so
// their walks share cache lines if they run on one XCD (one L2) at the same time:
// the walks of a launch start together and advance alike.  The workgroups of one
// band of detector rows are numbered in blocks of FWD_VIEWS views, in a block by
// pairs of column groups (8 columns), in a pair view by view; dispatch fills the
// eight XCDs round-robin, and each takes runs of FWD_RUN consecutive numbers.  A run
// covers 8 columns in 64 views: the planes its walks meet at one xi are
// about 100 z-columns.  Measured at 512^3 x 720, 616 x 480 detector, FP32: 48.6 ms, against
// 60.8 ms with all columns of a view together (every view read the volume anew:
// 414 GB beyond the L2); 256^3 x 360, 384 x 384: 4.79 against 5.50 ms; 192^3 x 180,
// 256 x 256: 0.85 against 0.99 ms.  Runs of 64 or 256, blocks of 64 views: within 1 %;
// pairs of one or four groups 1 to 3 % slower, one run per XCD 11 to 20 %.
constexpr unsigned FWD_PAIR = 2, FWD_VIEWS = 128, FWD_RUN = 128;

// The column group, view and band of workgroup w.  All products are at most f.nblocks,
// which a projection of less than 2^31 rays keeps below 2^31.
__host__ __device__ __forceinline__ void fwd_tile(const FwdGrid &f, unsigned w, int &cg, int &k, int &band)
{
    const unsigned n = (unsigned)f.nblocks, ncg = (unsigned)f.ncg, nviews = (unsigned)f.nviews;
    const unsigned full = n / (FWD_XCDS * FWD_RUN) * (FWD_XCDS * FWD_RUN);  // the rest keeps its order
    unsigned i = w < full ? (w / (FWD_XCDS * FWD_RUN) * FWD_XCDS + w % FWD_XCDS) * FWD_RUN + w / FWD_XCDS % FWD_RUN : w;
    band = (int)(i / (ncg * nviews));
    i -= (unsigned)band * (ncg * nviews);
    const unsigned block = ncg * (nviews < FWD_VIEWS ? nviews : FWD_VIEWS);
    const unsigned vb = i / block;
    i -= vb * block;
    const unsigned nv = nviews - vb * FWD_VIEWS < FWD_VIEWS ? nviews - vb * FWD_VIEWS : FWD_VIEWS;
    const unsigned pair = i / (FWD_PAIR * nv);
    i -= pair * (FWD_PAIR * nv);
    const unsigned np = ncg - pair * FWD_PAIR < FWD_PAIR ? ncg - pair * FWD_PAIR : FWD_PAIR;
    cg = (int)(pair * FWD_PAIR + (np == 2 ? i % 2 : 0));
    k = (int)(vb * FWD_VIEWS + (np == 2 ? i / 2 : i));
}

// The same for a volume read in its own layout in up to FWD_VIEWS_IN_PLACE views: the
// lanes of a wavefront (rows) share no cache line there but neighbouring columns do.
// Column group fastest, then view, then band; within 64 consecutive workgroups each XCD
// gets 8 neighbouring groups.  Measured (us, this order / the one above): 224 x 371 x 274,
// 13 views, FP64 4519 / 5128; 129 x 214 x 89, 9 views 259 / 371; 390 x 540 x 443, 4 views
// 4033 / 4595; 191 x 157 x 209, 61 views, bfloat16 1101 / 1299; with more views it loses:
// 214 x 91 x 142, 78 views 672 / 569; 262 x 143 x 400, 264 views 21490 / 15270.
constexpr int FWD_VIEWS_IN_PLACE = 64;
__host__ __device__ __forceinline__ void fwd_tile_in_place(const FwdGrid &f, unsigned w, int &cg, int &k, int &band)
{
    const unsigned full = (unsigned)f.nblocks & ~63u;
    const unsigned i = w < full ? (w & ~63u) + w % FWD_XCDS * 8 + w / FWD_XCDS % 8 : w;
    cg = (int)(i % (unsigned)f.ncg);
    const unsigned rest = i / (unsigned)f.ncg;
    k = (int)(rest % (unsigned)f.nviews);
    band = (int)(rest / (unsigned)f.nviews);
}

// forward_block runs workgroup w (0 <= w < fwd_grid(g, R).nblocks) of the
// projection of one volume; R rows per lane.  Its partial sum goes to
// partials[w].  A ray is walked whole (FWD_WHOLE, workgroups of 4 wavefronts, one
// per column), or in FWD_PARTS shares whose sums are added pairwise: at once by 16
// wavefronts (FWD_DIVIDED: wavefronts 4 i + c take share i of column c), or one after
// the other by 4 (FWD_IN_TURN), with the same result.  shares: LDS for
// FWD_PARTS x FWD_COLS x R x 64 sums (FWD_DIVIDED).  ZFAST: vol_z is given.
enum FwdWalk { FWD_WHOLE = 0, FWD_DIVIDED, FWD_IN_TURN };
template <typename TV, typename TP, int EPI, int R, int WALK, bool ZFAST>
__device__ __forceinline__ void forward_block(const GeoDev &g, int64_t w, const TV *__restrict__ vol,
                                              const TV *__restrict__ vol_z, TP *__restrict__ out,
                                              const TP *__restrict__ aux, const Scalars *__restrict__ sc,
                                              double *__restrict__ partials, acc_t<TV> *shares)
{
    constexpr int FWD_ROWS = 64 * R;
    const FwdGrid fg = fwd_grid(g, R);
    int cg, k, band;
    if (!ZFAST && WALK == FWD_WHOLE && g.nviews <= FWD_VIEWS_IN_PLACE)
        fwd_tile_in_place(fg, (unsigned)w, cg, k, band);
    else
        fwd_tile(fg, (unsigned)w, cg, k, band);
    // the wavefront's column, made provably uniform so that the in-plane walk
    // (a function of the column) runs on scalar registers and branches
    const int wave = __builtin_amdgcn_readfirstlane((int)(__builtin_amdgcn_workitem_id_x() >> 6));
    const int iu = cg * FWD_COLS + wave % FWD_COLS;
    const int lane = (int)(__builtin_amdgcn_workitem_id_x() & 63);
    ViewParam vp = g.views[k];
    vp.dom = __builtin_amdgcn_readfirstlane(vp.dom);  // uniform: the volume's base and strides follow it

    int nxi, neta, sxi, seta, sz;
    float hxi, heta;
    const TV *base;
    if (vp.dom == 0) {  // xi = x, eta = y
        nxi = g.nx; neta = g.ny; hxi = g.hx; heta = g.hy;
        if (ZFAST) { base = vol_z; sz = 1; sxi = g.nz; seta = g.nx * g.nz; }
        else { base = vol; sz = g.nx * g.ny; sxi = 1; seta = g.nx; }
    } else {            // xi = y, eta = x
        nxi = g.ny; neta = g.nx; hxi = g.hy; heta = g.hx;
        if (ZFAST) { base = vol_z; sz = 1; sxi = g.nx * g.nz; seta = g.nz; }
        else { base = vol; sz = g.nx * g.ny; sxi = g.nx; seta = 1; }
    }

    // lane rows: band * FWD_ROWS + lane + 64 r
    using A = acc_t<TV>;
    float zc[R], czr[R], Ls[R];
    A p[R];
    bool ok[R];
    const bool col_ok = iu < g.nu;
    ColParam cp{};
    if (col_ok) cp = g.cols[(size_t)k * g.nu + iu];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int iv = band * FWD_ROWS + lane + 64 * r;
        ok[r] = col_ok && iv < g.nv;
        const RowParam rp = ok[r] ? g.rows[iv] : RowParam{0.0f, 0.0f};
        zc[r] = zeta_centre(rp.qz, cp.tcv, g.zc);
        czr[r] = zeta_inv_slope(rp.inv_qz, cp.kz);
        Ls[r] = ray_length_per_xi(cp.lxy2, rp.qz, cp.gp);
        if (!ok[r]) czr[r] = 1.0f, zc[r] = 3.0e30f;  // far outside: an inert ray
    }
    // this wavefront's share of the walk, or all of them in turn
    auto walk = [&](A (&s)[R], int part, int of) {
        if (!col_ok) {
#pragma unroll
            for (int r = 0; r < R; ++r) s[r] = 0;
        } else if constexpr (ZFAST) {
            trace_rays<TV, R, 1>(base, sxi, seta, sz, nxi, neta, g.nz, hxi, heta, g.hz, cp.eta_c, cp.inv_a, cp.a, zc,
                                 czr, s, part, of);
        } else {
            trace_rays<TV, R, 0>(base, sxi, seta, sz, nxi, neta, g.nz, hxi, heta, g.hz, cp.eta_c, cp.inv_a, cp.a, zc,
                                 czr, s, part, of);
        }
    };
    A s[R];
    if constexpr (WALK == FWD_WHOLE) {
        walk(s, 0, 1);
    } else if constexpr (WALK == FWD_DIVIDED) {
        walk(s, wave / FWD_COLS, FWD_PARTS);
#pragma unroll
        for (int r = 0; r < R; ++r) shares[(wave * R + r) * 64 + lane] = s[r];
        __syncthreads();
        if (wave < FWD_COLS) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                A v[FWD_PARTS];
#pragma unroll
                for (int q = 0; q < FWD_PARTS; ++q) v[q] = shares[((q * FWD_COLS + wave) * R + r) * 64 + lane];
                s[r] = (v[0] + v[1]) + (v[2] + v[3]);
            }
        }
    } else {
        // (share 1 added to share 0, share 3 to share 2, and the two sums)
        A pair[R];
        for (int q = 0; q < FWD_PARTS; ++q) {
            A t[R];
            walk(t, q, FWD_PARTS);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const A both = (q & 1) ? pair[r] + t[r] : t[r];
                s[r] = q == 3 ? s[r] + both : (q < 2 ? both : s[r]);
                pair[r] = both;
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) p[r] = (A)Ls[r] * s[r];
    double sq = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!ok[r] || (WALK == FWD_DIVIDED && wave >= FWD_COLS)) continue;
        const int iv = band * FWD_ROWS + lane + 64 * r;
        const size_t ray = ((size_t)k * g.nv + iv) * g.nu + iu;
        sq += fwd_store<TP, EPI, A>(out, aux, sc, ray, p[r]);
    }
    if (EPI != FWD_PLAIN) {
        const double bs = fwd_block_sum(sq);
        if (__builtin_amdgcn_workitem_id_x() == 0) partials[w] = bs;
    }
}

// Registers with four rows: 63 with the z-fastest copy (8 wavefronts per SIMD), 65 with a
// solver's epilogue and 70 to 72 in place (7); fewer rows need fewer.
template <typename TV, typename TP, int EPI, int R, bool ZFAST>
__global__ __launch_bounds__(256, sizeof(acc_t<TV>) != 4 ? 1 : (R > 3 ? 7 : 8)) void k_forward(
    GeoDev g, const TV *__restrict__ vol, const TV *__restrict__ vol_z, TP *__restrict__ out, const TP *__restrict__ aux,
    const Scalars *__restrict__ sc, double *__restrict__ partials, const int *__restrict__ skip)
{
    if (skip && *skip) return;
    forward_block<TV, TP, EPI, R, FWD_WHOLE, ZFAST>(g, __builtin_amdgcn_workgroup_id_x(), vol, vol_z, out, aux, sc, partials,
                                                    nullptr);
}

// The walk of every ray divided among FWD_PARTS wavefronts.
template <typename TV, typename TP, int EPI, int R, bool ZFAST>
__global__ __launch_bounds__(256 * FWD_PARTS) void k_forward_divided(
    GeoDev g, const TV *__restrict__ vol, const TV *__restrict__ vol_z, TP *__restrict__ out, const TP *__restrict__ aux,
    const Scalars *__restrict__ sc, double *__restrict__ partials, const int *__restrict__ skip)
{
    __shared__ acc_t<TV> shares[FWD_PARTS * FWD_COLS * R * 64];
    if (skip && *skip) return;
    forward_block<TV, TP, EPI, R, FWD_DIVIDED, ZFAST>(g, __builtin_amdgcn_workgroup_id_x(), vol, vol_z, out, aux, sc, partials,
                                                      shares);
}

// The launch of a forward projection with R rows per lane; divided (R <= 2): see FwdPlan.
template <typename TV, typename TP, int EPI, int R, bool ZFAST>
static hipError_t launch_forward_epi(const GeoDev &g, bool divided, const TV *vol, const TV *vol_z, TP *out, const TP *aux,
                                     const Scalars *sc, double *partials, const int *skip, hipStream_t st)
{
    const dim3 grid((unsigned)fwd_grid(g, R).nblocks);
    if constexpr (R <= 2) {
        if (divided) {
            hipLaunchKernelGGL((k_forward_divided<TV, TP, EPI, R, ZFAST>), grid, dim3(256 * FWD_PARTS), 0, st, g, vol, vol_z,
                               out, aux, sc, partials, skip);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_forward<TV, TP, EPI, R, ZFAST>), grid, dim3(256), 0, st, g, vol, vol_z, out, aux, sc, partials,
                       skip);
    return hipGetLastError();
}

// The forms that are called: plain projections and b - A x with and without the z-fastest
// copy, the solvers' directions, which have it, in the storage of the projections, and b - A x
// of the single-precision iterate (double storage: plain projections only).
template <typename TV, typename TP, int R>
hipError_t launch_forward_rows(const GeoDev &g, bool divided, const TV *vol, const TV *vol_z, TP *out, const TP *aux,
                               int epi, const Scalars *sc, double *partials, const int *skip, hipStream_t st)
{
    if constexpr (std::is_same<TV, TP>::value) {
        if (epi == FWD_PLAIN)
            return vol_z ? launch_forward_epi<TV, TP, FWD_PLAIN, R, true>(g, divided, vol, vol_z, out, aux, sc, partials, skip, st)
                         : launch_forward_epi<TV, TP, FWD_PLAIN, R, false>(g, divided, vol, vol_z, out, aux, sc, partials, skip, st);
        if constexpr (!std::is_same<TV, double>::value) {
            if (epi == FWD_NORM && vol_z)
                return launch_forward_epi<TV, TP, FWD_NORM, R, true>(g, divided, vol, vol_z, out, aux, sc, partials, skip, st);
            if (epi == FWD_LSQR && vol_z)
                return launch_forward_epi<TV, TP, FWD_LSQR, R, true>(g, divided, vol, vol_z, out, aux, sc, partials, skip, st);
        }
    }
    if constexpr (std::is_same<TV, float>::value) {
        if (epi == FWD_BMINUS)
            return vol_z ? launch_forward_epi<TV, TP, FWD_BMINUS, R, true>(g, divided, vol, vol_z, out, aux, sc, partials, skip, st)
                         : launch_forward_epi<TV, TP, FWD_BMINUS, R, false>(g, divided, vol, vol_z, out, aux, sc, partials, skip, st);
    }
    return hipErrorInvalidValue;
}

// every storage combination of launch_forward_rows with R rows per lane
#define KCT_FORWARD_ROWS(R)                                                                                             \
    KCT_FORWARD_INST(float, float, R)                                                                                  \
    KCT_FORWARD_INST(bf16, bf16, R)                                                                                    \
    KCT_FORWARD_INST(_Float16, _Float16, R)                                                                            \
    KCT_FORWARD_INST(float, bf16, R)                                                                                   \
    KCT_FORWARD_INST(float, _Float16, R)                                                                               \
    KCT_FORWARD_INST(double, double, R)
#define KCT_FORWARD_INST(TV, TP, R)                                                                                     \
    template hipError_t launch_forward_rows<TV, TP, R>(const GeoDev &, bool, const TV *, const TV *, TP *, const TP *, int, \
                                                       const Scalars *, double *, const int *, hipStream_t);

}  // namespace kct
