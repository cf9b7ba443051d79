// kct_wave.h -- the wave form of the backprojection: one wavefront takes a brick
// of WX x WY voxel columns, TZB deep, and a subset of the views.  Per view it
// bounds the brick's detector shadow, stages it in an LDS region of its own and
// gathers from it (kct_gather.h), with no workgroup barrier in the view loop.
//
// The 16 x 16 column bricks of backproject.hip need about 4000 workgroups to fill
// the chip and one pass through all views for each; volumes up to 192^3 have
// 4 to 1728 of them.  Here a brick has a quarter of the columns, its depth
// follows the shadow (so that one view's shadow is one staged chunk also where
// a voxel spans several pixels), and the views are dealt to up to 16 subsets.
//
// Bounded by VALU issue and, where a voxel spans more than a pixel, by the LDS reads of
// the records; a quarter to a third of its instructions stage the shadow.  Bricks up
// to 16 deep are staged in split records (kct_gather.h), which let a chunk hold 640 of
// them in less LDS than 448 whole ones.  Measured (one backprojection, 16 x 16 x 16
// workgroup bricks -> this form with whole records -> split): 64^3 x 90 views, 96 x 96
// detector 1260 -> 96 -> 87 us; 96^3 x 186, 218 x 218 4170 -> 839 -> 640 us; 64^3 x 199,
// 274 x 274 (four pixels per voxel) 22.4 -> 1.42 -> 1.06 ms; 192^3 x 180, 256 x 256
// 2.38 -> 1.89 -> 1.61 ms; 256^3 x 360, 384 x 384 10.5 -> 8.6 (bricks) -> 8.2 ms; whole
// records: 128^3 x 720, 154 x 120 3.06 -> 1.39 ms.  With the sums' pointers read late
// (BwdOut) 78 us, 0.58 ms, 1.05 ms, 1.61 ms, 8.04 ms and 1.32 ms.
#pragma once

#include "kct_epilogue.h"
#include "kct_gather.h"
#include "kct_internal.h"
#include "kct_weights.h"

namespace kct {

constexpr int WX = 8, WY = 8;    // voxel columns of a brick: one per lane
constexpr int W_GROUPS = 4;      // the view subsets are added within groups, then the groups
// Staged records of a chunk, its zero row included: room for the shadow of the deepest brick
// against wavefronts per CU.  Measured (us, 576 / 640 / 720): 64^3 x 199, 274 x 274 1152 / 1098 / 1076;
// 96^3 x 186 667 / 654 / 786; 192^3 x 180 1639 / 1646 / 1804; 192^3 x 120 at 2.2 pixels per voxel
// 3080 / 2920 / 3126.
constexpr int W_CAP = 640;
constexpr int W_CAP_FULL = 448;  // the same for 16-byte records
constexpr int W_NHMAX = 3;

// Detector columns held in registers at once: shallow bricks are those of wide
// shadows, where a lane meets three and more columns.
__host__ __device__ constexpr int wave_nh(int tzb) { return tzb <= 8 ? 3 : 2; }

constexpr int W_SUMS = 8;        // voxels per lane whose partial sums pass through LDS at once

__host__ __device__ constexpr int wave_cap(bool split) { return split ? W_CAP : W_CAP_FULL; }
// Most columns of a chunk (whole records: the deepest bricks, whose shadows are narrow; with
// more, five workgroups of the batched form would not fit the LDS).
__host__ __device__ constexpr int wave_cols(bool split) { return split ? 48 : 32; }
__host__ __device__ constexpr int wave_rows(bool split) { return wave_cap(split) / 8; }  // most rows of a chunk, with its zero row

// Records of one wavefront's staging region: the chunk and the spare records
// that add_row may read.
__host__ __device__ constexpr int wave_region(bool split) { return wave_cap(split) + W_NHMAX - 1; }

// LDS bytes of a workgroup of `waves` wavefronts: staging regions, columns and row
// factors.
template <typename A, bool SPLIT> __host__ __device__ constexpr size_t wave_lds_bytes(int waves)
{
    return (size_t)waves * (wave_region(SPLIT) * sizeof(PixStage<A, SPLIT>) + wave_cols(SPLIT) * sizeof(ColStage) +
                            (SPLIT ? wave_rows(SPLIT) * sizeof(float) : 0));
}

// Orders one wavefront's LDS writes before its later reads, and its reads
// before later writes (the LDS serves a wavefront in order; this keeps the
// compiler from reordering them).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The element of type E at byte offset off from base.
template <typename E> __device__ __forceinline__ const E *byte_at(const void *base, unsigned off)
{
    return reinterpret_cast<const E *>(static_cast<const char *>(base) + off);
}

// Where a backprojection's sums go, needed after the view loop only.  A kernel takes it
// as its first argument and reads it from the argument segment after the loop
// (late_out): kept through the loop, the five pointers take ten of the scalar registers
// that the loop is short of, and what is then spilled to vector registers costs a
// wavefront per SIMD (16-deep wave form of the solvers, 256^3 x 360 9.2 ms against 8.1).
template <typename T> struct BwdOut {
    T *out, *out_z;
    const Scalars *sc;
    double *partials;
    const float *aux;
};

// The running kernel's first argument, read where this stands.
template <typename T> __device__ __forceinline__ BwdOut<T> late_out()
{
    typedef const __attribute__((address_space(4))) BwdOut<T> *segment;
    segment a = (segment)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return BwdOut<T>{a->out, a->out_z, a->sc, a->partials, a->aux};
}

// Brick w (0 <= w < nbx * nby * nbz) of the backprojection, by a workgroup of `waves`
// wavefronts, the views dealt to `sets` subsets (1, 2 or a multiple of W_GROUPS): views
// s, s + sets, ... are subset s.  With subs = sets / waves (at least 1), wavefront v takes
// the subsets v * subs, v * subs + 1, ... in turn, so `waves` is sets or a divisor of it
// (or above it, those beyond without a view).  A voxel's partial sums are added in
// order within each of W_GROUPS groups of neighbouring subsets (one subset each where
// there are fewer), and the groups pairwise, so the sum depends on `sets` alone; the
// squares of a layer of voxels are added first, then the layers in order, so the
// partial sum of squares, which goes to the partials' [w], depends on `sets` alone as
// well.  lds: wave_lds_bytes(waves) bytes, 16-byte aligned.  BATCH: waves is
// W_GROUPS; else it is sets.  late(): the BwdOut, after the view loop.
template <typename T, int EPI, int TZB, bool BATCH, typename Late>
__device__ __forceinline__ void backward_wave_block(const GeoDev &g, int w, const T *__restrict__ proj, int nbx, int nby,
                                                    int nbz, int waves, int sets, void *lds, Late late)
{
    using A = acc_t<T>;
    constexpr bool SQ = EPI == BWD_DIAG || EPI == BWD_DIAG_INV;  // squared weights, e not read
    constexpr bool SPLIT = split_records<A>(TZB);
    constexpr int CAP = wave_cap(SPLIT), ROWS = wave_rows(SPLIT), REGION = wave_region(SPLIT), COLS = wave_cols(SPLIT),
                  NCOL = wave_nh(TZB);
    using Rec = PixStage<A, SPLIT>;
    static_assert(sizeof(A) * W_SUMS * 64 <= sizeof(Rec) * REGION, "the partial sums fit a staging region");
    Rec *s_all = static_cast<Rec *>(lds);
    ColStage *c_all = reinterpret_cast<ColStage *>(s_all + waves * REGION);
    double *layer_sq = reinterpret_cast<double *>(c_all);  // once the columns are no longer read
    static_assert(sizeof(double) * TZB <= sizeof(ColStage) * COLS, "a layer's sum of squares each");
    const int wave = __builtin_amdgcn_readfirstlane((int)(__builtin_amdgcn_workitem_id_x() >> 6));
    const int lane = (int)(__builtin_amdgcn_workitem_id_x() & 63);
    Rec *s_pix = s_all + wave * REGION;
    ColStage *s_col = c_all + wave * COLS;
    float *s_row = reinterpret_cast<float *>(c_all + waves * COLS) + wave * ROWS;  // used when SPLIT

    // XCD-aware brick assignment (see backproject.hip)
    constexpr int XCDS = 8;
    const int nb = nbx * nby * nbz;
    const int b = (nb % XCDS == 0) ? (w % XCDS) * (nb / XCDS) + w / XCDS : w;
    const int bx = b % nbx, by = (b / nbx) % nby, bz = b / (nbx * nby);
    const int ix = bx * WX + lane % WX, iy = by * WY + lane / WX;
    const int iz0 = bz * TZB;
    const int nzb = g.nz - iz0 < TZB ? g.nz - iz0 : TZB;
    const bool valid = ix < g.nx && iy < g.ny;
    // half extents and centre of the brick's square, heights of its lowest and highest plane [mm]
    const int cnx = g.nx - bx * WX < WX ? g.nx - bx * WX : WX, cny = g.ny - by * WY < WY ? g.ny - by * WY : WY;
    const float ex = 0.5f * (float)cnx * g.vx, ey = 0.5f * (float)cny * g.vy;
    const float xc = g.x0 + (float)(bx * WX) * g.vx + ex, yc = g.y0 + (float)(by * WY) * g.vy + ey;
    const float wz0 = g.z0 + (float)iz0 * g.vz, wz1 = g.z0 + (float)(iz0 + nzb) * g.vz;

    constexpr bool MANY = BATCH && TZB < TZ_DEEP;  // a wavefront may take several subsets
    A acc[TZB], sum[MANY ? TZB : 1];
#pragma unroll
    for (int j = 0; j < TZB; ++j) acc[j] = 0;

    const int subs = MANY && sets > waves ? sets / waves : 1;
    for (int turn = 0; turn < subs; ++turn) {
        for (int k = !BATCH ? wave : (wave < sets ? wave * subs + turn : g.nviews); k < g.nviews; k += BATCH ? sets : waves) {
            const ViewParam vp = g.views[k];
            // 1. shadow of the brick, as voxel_columns bounds one voxel's: its
            //    detector columns around the image of its centre, its rows from the
            //    heights of its planes at its square's least and greatest depth
            int u0, u1, v0, v1;
            {
                const float dn = __builtin_fmaf(ex, fabsf(vp.s), ey * fabsf(vp.c));  // half extent along e_u
                const float dd = __builtin_fmaf(ex, fabsf(vp.c), ey * fabsf(vp.s));  // and in depth
                const float dx = xc - vp.sx, dy = yc - vp.sy;
                const float num = __builtin_fmaf(vp.c, dy, -vp.s * dx);
                const float den = __builtin_fmaf(-vp.c, dx, -vp.s * dy);
                const float inv = rcp_approx(den), rmax = rcp_approx(den - dd), rmin = rcp_approx(den + dd);
                const float fc = __builtin_fmaf(num * inv, g.ku, g.fu0);
                const float hc = __builtin_fmaf(__builtin_fmaf(dd * fabsf(num), inv, dn) * rmax, g.ku, 0.01f);
                const float p0 = wz0 * rmin, p1 = wz0 * rmax, p2 = wz1 * rmin, p3 = wz1 * rmax;
                const float zlo = fminf(fminf(p0, p1), fminf(p2, p3)), zhi = fmaxf(fmaxf(p0, p1), fmaxf(p2, p3));
                const int a0 = (int)ceilf(fc - hc), a1 = (int)floorf(fc + hc);
                const int b0 = (int)ceilf(__builtin_fmaf(zlo, g.kv, g.fv0) - 0.01f);
                const int b1 = (int)floorf(__builtin_fmaf(zhi, g.kv, g.fv0) + 0.01f);
                u0 = __builtin_amdgcn_readfirstlane(a0 < 0 ? 0 : a0);
                u1 = __builtin_amdgcn_readfirstlane(a1 > g.nu - 1 ? g.nu - 1 : a1);
                v0 = __builtin_amdgcn_readfirstlane(b0 < 0 ? 0 : b0);
                v1 = __builtin_amdgcn_readfirstlane(b1 > g.nv - 1 ? g.nv - 1 : b1);
            }
            const T *pk = SQ ? proj : proj + (size_t)k * g.nv * g.nu;  // not read when SQ
            const ColParam *ck = g.cols + (size_t)k * g.nu;
            // chunks of at most CAP records with the zero row, COLS columns, and
            // rows that leave room for 8 columns; typical bricks need one chunk
            constexpr int RMAX = ROWS - 1;
            for (int cv0 = v0; cv0 <= v1; cv0 += RMAX) {
                const int nrow = v1 - cv0 + 1 < RMAX ? v1 - cv0 + 1 : RMAX;
                int cmax = COLS;
                if ((nrow + 1) * cmax > CAP) {
                    // CAP / (nrow + 1) through a reciprocal, one less where that rounds up
                    cmax = __builtin_amdgcn_readfirstlane((int)((float)CAP * __builtin_amdgcn_rcpf((float)(nrow + 1)) + 0.01f));
                    if ((nrow + 1) * cmax > CAP) --cmax;
                }
                for (int cu0 = u0; cu0 <= u1; cu0 += cmax) {
                    const int ncol = u1 - cu0 + 1 < cmax ? u1 - cu0 + 1 : cmax;
                    // 2. stage the chunk: lane t keeps column t % ncol and takes the rows
                    //    t / ncol, + step, ... of it (the division through a reciprocal:
                    //    (t + 0.5) / ncol lies at least 0.5 / ncol >= 0.01 from an integer,
                    //    the product's rounding below 1e-4)
                    {
                        const float rn = __builtin_amdgcn_rcpf((float)ncol);
                        const int step = __builtin_amdgcn_readfirstlane((int)(64.5f * rn));
                        const int r0 = (int)(((float)lane + 0.5f) * rn), c = lane - r0 * ncol;
                        if (r0 < step) {
                            const ColParam cp = *byte_at<ColParam>(ck, (unsigned)(cu0 + c) * (unsigned)sizeof(ColParam));
                            if (r0 == 0) s_col[c] = stage_column(g, vp.dom, cp);
                            unsigned pix = ((unsigned)(cv0 + r0) * (unsigned)g.nu + (unsigned)(cu0 + c)) * (unsigned)sizeof(T);
                            unsigned row = (unsigned)(cv0 + r0) * (unsigned)sizeof(RowParam);
                            Rec *rec = s_pix + (r0 * ncol + c);
                            for (int r = r0; r < nrow; r += step) {
                                const A ev = SQ ? (A)0 : to_acc(*byte_at<T>(pk, pix));
                                *rec = stage_pixel<A, SQ, SPLIT>(cp, *byte_at<RowParam>(g.rows, row), ev);
                                pix += (unsigned)(step * g.nu) * (unsigned)sizeof(T);
                                row += (unsigned)step * (unsigned)sizeof(RowParam);
                                rec += step * ncol;
                            }
                            if (r0 == 0) s_pix[nrow * ncol + c] = zero_pixel<A, SPLIT>();
                        }
                    }
                    if constexpr (SPLIT)
                        for (int r = lane; r <= nrow; r += 64) s_row[r] = r < nrow ? g.rows[cv0 + r].s_inv : 0.0f;
                    wave_lds_order();
                    // 3. gather (the lane's column indices laundered per chunk: what is
                    //    derived from them is recomputed instead of kept through the view loop)
                    int ixv = ix, iyv = iy;
                    asm volatile("" : "+v"(ixv), "+v"(iyv));
                    if (valid)
                        gather_chunk<A, SQ, 0, NCOL, true>(g, vp, ixv, iyv, iz0, s_pix, s_col, s_row, cu0, ncol, cv0, nrow, nzb, acc, ncol);
                    wave_lds_order();
                }
            }
        }
        if (MANY) {
#pragma unroll
            for (int j = 0; j < TZB; ++j) {
                sum[MANY ? j : 0] = turn == 0 ? acc[j] : sum[MANY ? j : 0] + acc[j];
                acc[j] = 0;
            }
        }
    }

    // every voxel's partial sums through LDS, W_SUMS voxels of each lane at a time:
    // in order within a group, then the groups
    const BwdOut<T> o = late();
    A *mine = reinterpret_cast<A *>(s_pix);
    const int per = waves > W_GROUPS ? waves / W_GROUPS : 1;
#pragma unroll
    for (int j0 = 0; j0 < TZB; j0 += W_SUMS) {
        if (j0 > 0) __syncthreads();
#pragma unroll
        for (int j = j0; j < j0 + W_SUMS && j < TZB; ++j)
            mine[(j - j0) * 64 + lane] = MANY ? sum[MANY ? j : 0] : acc[j];
        __syncthreads();
        const int jend = nzb < j0 + W_SUMS ? nzb : j0 + W_SUMS;
        for (int j = j0 + wave; j < jend; j += waves) {
            const int at = (j - j0) * 64 + lane;
            A v[W_GROUPS];
#pragma unroll
            for (int q = 0; q < W_GROUPS; ++q) {
                v[q] = 0;
                if (q * per >= waves) continue;
                v[q] = reinterpret_cast<const A *>(s_all + q * per * REGION)[at];
                for (int i = 1; i < per; ++i) v[q] += reinterpret_cast<const A *>(s_all + (q * per + i) * REGION)[at];
            }
            double sq = 0.0;
            if (valid) {
                const int iz = iz0 + j;
                const size_t vox = ((size_t)iz * g.ny + iy) * g.nx + ix;
                sq = bwd_store<T, EPI, A>(o.out, o.out_z, o.sc, o.aux, vox, ((size_t)iy * g.nx + ix) * g.nz + iz,
                                          (v[0] + v[1]) + (v[2] + v[3]));
            }
            if (bwd_has_partials<EPI>()) {
                for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
                if (lane == 0) layer_sq[j] = sq;
            }
        }
    }
    if (bwd_has_partials<EPI>()) {
        __syncthreads();
        if (__builtin_amdgcn_workitem_id_x() == 0) {
            double r = layer_sq[0];
            for (int j = 1; j < nzb; ++j) r += layer_sq[j];
            o.partials[w] = r;
        }
    }
}

}  // namespace kct
