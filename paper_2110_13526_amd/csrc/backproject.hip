// backproject.hip -- r = A^T e (Section 2, Eq. 2) as a voxel-driven gather on
// gfx950: one workgroup per brick of BX x BY x TZ voxels, all views in one
// launch, the brick's detector shadow staged in LDS per view (see
// kct_gather.h).  Every voxel is written once by the lane that owns it; no
// atomics; bitwise reproducible.
//
// Workgroups are assigned to bricks so that each of the eight XCDs (which fill
// round-robin in dispatch order) owns a contiguous range of bricks: bricks that
// neighbour each other share most of their detector shadow, so the staged
// projection values are reused from the XCD's own L2.
#include <cmath>
#include <type_traits>

#include "kct_batch.h"
#include "kct_epilogue.h"
#include "kct_gather.h"
#include "kct_internal.h"
#include "kct_wave.h"
#include "kct_weights.h"

namespace kct {

constexpr int NXCD = 8;
static_assert(BX == 16 && BY == 16, "the shadow table (ShadowParam) is built for columns of 16 x 16 voxels");

__device__ __forceinline__ double bwd_block_sum(double v)
{
    __shared__ double red[4];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((__builtin_amdgcn_workitem_id_x() & 63) == 0) red[__builtin_amdgcn_workitem_id_x() >> 6] = v;
    __syncthreads();
    double r = 0.0;
    if (__builtin_amdgcn_workitem_id_x() == 0) r = (red[0] + red[1]) + (red[2] + red[3]);
    return r;
}

// backward_block runs workgroup w (0 <= w < nbx * nby * nbz) of the
// backprojection into one volume; its partial sum goes to the partials' [w].  late(): the
// BwdOut, after the view loop (see there).
// s_pix / s_col / s_row: LDS for ch_rows(TZB) x CHC staged pixels (plus a zero row and a
// spare record), CHC columns and ch_rows(TZB) + 1 rows.
template <typename T, int EPI, int TZB, int CHC, typename Late>
__device__ __forceinline__ void backward_block(const GeoDev &g, int w, const T *__restrict__ proj, int nbx, int nby, int nbz,
                                               PixStage<acc_t<T>, split_records<acc_t<T>>(TZB)> *s_pix, ColStage *s_col,
                                               float *s_row, Late late)
{
    using A = acc_t<T>;
    constexpr int CHR = ch_rows(TZB);  // staged rows per chunk
    constexpr bool SPLIT = split_records<A>(TZB);
    constexpr bool SQ = EPI == BWD_DIAG || EPI == BWD_DIAG_INV;  // squared weights, e not read

    // XCD-aware brick assignment
    const int nb = nbx * nby * nbz;
    const int b = (nb % NXCD == 0) ? (w % NXCD) * (nb / NXCD) + w / NXCD : w;
    const int bx = b % nbx, by = (b / nbx) % nby, bz = b / (nbx * nby);
    const int ix = bx * BX + (int)(__builtin_amdgcn_workitem_id_x() % BX);
    const int iy = by * BY + (int)(__builtin_amdgcn_workitem_id_x() / BX);
    const int iz0 = bz * TZB;
    const int nzb = g.nz - iz0 < TZB ? g.nz - iz0 : TZB;
    const bool valid = ix < g.nx && iy < g.ny;

    // the brick's column in the shadow table, and its lowest and highest plane
    // (heights above the source plane, mm)
    const int sbi = __builtin_amdgcn_readfirstlane(by * g.sbx + bx);  // uniform: the table row stays scalar
    const size_t sbxy = (size_t)g.sbx * g.sby;
    const float wz0 = g.z0 + (float)iz0 * g.vz, wz1 = g.z0 + (float)(iz0 + nzb) * g.vz;

    A acc[TZB];
#pragma unroll
    for (int j = 0; j < TZB; ++j) acc[j] = 0;

    for (int k = 0; k < g.nviews; ++k) {
        const ViewParam vp = g.views[k];
        // 1. shadow of the brick: its column's detector columns from the table
        //    (uniform: scalar loads), its rows from the heights of its lowest and
        //    highest plane seen at the column's extreme inverse depths, widened
        //    by 0.01 row against rounding
        int u0, u1, v0, v1;
        {
            const ShadowParam sh = g.shadows[(size_t)k * sbxy + sbi];
            u0 = sh.u0;
            u1 = sh.u1;
            const float p0 = wz0 * sh.rmin, p1 = wz0 * sh.rmax, p2 = wz1 * sh.rmin, p3 = wz1 * sh.rmax;
            const float zlo = fminf(fminf(p0, p1), fminf(p2, p3)), zhi = fmaxf(fmaxf(p0, p1), fmaxf(p2, p3));
            const int b0 = (int)ceilf(__builtin_fmaf(zlo, g.kv, g.fv0) - 0.01f);
            const int b1 = (int)floorf(__builtin_fmaf(zhi, g.kv, g.fv0) + 0.01f);
            v0 = __builtin_amdgcn_readfirstlane(b0 < 0 ? 0 : b0);
            v1 = __builtin_amdgcn_readfirstlane(b1 > g.nv - 1 ? g.nv - 1 : b1);
        }
        const T *pk = SQ ? proj : proj + (size_t)k * g.nv * g.nu;  // not read when SQ
        const ColParam *ck = g.cols + (size_t)k * g.nu;
        for (int cu0 = u0; cu0 <= u1; cu0 += CHC) {
            const int ncol = u1 - cu0 + 1 < CHC ? u1 - cu0 + 1 : CHC;
            for (int cv0 = v0; cv0 <= v1; cv0 += CHR) {
                const int nrow = v1 - cv0 + 1 < CHR ? v1 - cv0 + 1 : CHR;
                // the thread index read here (an empty asm keeps the compiler from
                // hoisting what is derived from it out of the brick loops of the
                // persistent form, where it spilled)
                unsigned tid = __builtin_amdgcn_workitem_id_x();
                asm volatile("" : "+v"(tid));
                // 2. stage the chunk: per pixel the z-parameters of its ray and L * e,
                //    per column the in-plane parameters.  Thread t keeps column
                //    t % ncol (its ray parameters are read once per chunk) and takes
                //    the rows t / ncol, + step, ... of it; the threads past the last
                //    whole step of rows have nothing to stage.
                {
                    // tid / ncol through a reciprocal: (t + 0.5) / ncol lies at least
                    // 0.5 / ncol >= 0.01 from an integer, the product's rounding below 1e-4
                    const float rn = __builtin_amdgcn_rcpf((float)ncol);
                    const int step = __builtin_amdgcn_readfirstlane((int)(256.5f * rn));
                    const int r0 = (int)(((float)tid + 0.5f) * rn), c = (int)tid - r0 * ncol;
                    if (r0 < step) {
                        // all addressed as a uniform base plus a 32-bit byte offset (one
                        // view's projection values span < 2^31 bytes, the row parameters
                        // and one view's column parameters < 2^32: a detector has < 2^28
                        // pixels and < 2^27 columns)
                        const ColParam cp = *byte_at<ColParam>(ck, (unsigned)(cu0 + c) * (unsigned)sizeof(ColParam));
                        if (r0 == 0) s_col[c] = stage_column(g, vp.dom, cp);
                        unsigned pix = ((unsigned)(cv0 + r0) * (unsigned)g.nu + (unsigned)(cu0 + c)) * (unsigned)sizeof(T);
                        unsigned row = (unsigned)(cv0 + r0) * (unsigned)sizeof(RowParam);
                        PixStage<A, SPLIT> *rec = s_pix + (r0 * CHC + c);
                        for (int r = r0; r < nrow; r += step) {
                            const A ev = SQ ? (A)0 : to_acc(*byte_at<T>(pk, pix));
                            *rec = stage_pixel<A, SQ, SPLIT>(cp, *byte_at<RowParam>(g.rows, row), ev);
                            pix += (unsigned)(step * g.nu) * (unsigned)sizeof(T);
                            row += (unsigned)step * (unsigned)sizeof(RowParam);
                            rec += step * CHC;
                        }
                    }
                }
                // a zero row after the chunk's last: the gather reads a voxel's first
                // candidate row without a branch, and this one has weight 0 for any voxel
                if (tid < ncol) s_pix[nrow * CHC + tid] = zero_pixel<A, SPLIT>();
                if (SPLIT && tid <= nrow) s_row[tid] = tid < nrow ? g.rows[cv0 + tid].s_inv : 0.0f;
                __syncthreads();
                // 3. gather
                // the lane's column indices laundered per chunk: the few values derived
                // from them are recomputed here instead of being kept live (and spilled)
                // through the view loop
                int ixv = ix, iyv = iy;
                asm volatile("" : "+v"(ixv), "+v"(iyv));
                if (valid)
                    gather_chunk<A, SQ, CHC, NH, (TZB < TZ_DEEP)>(g, vp, ixv, iyv, iz0, s_pix, s_col, s_row, cu0, ncol, cv0, nrow, nzb, acc);
                __syncthreads();
            }
        }
    }

    const BwdOut<T> o = late();
    double sq = 0.0;
    if (valid) {
#pragma unroll
        for (int j = 0; j < TZB; ++j) {
            if (j >= nzb) continue;
            const int iz = iz0 + j;
            const size_t vox = ((size_t)iz * g.ny + iy) * g.nx + ix;
            sq += bwd_store<T, EPI, A>(o.out, o.out_z, o.sc, o.aux, vox, ((size_t)iy * g.nx + ix) * g.nz + iz, acc[j]);
        }
    }
    if (bwd_has_partials<EPI>()) {
        const double bs = bwd_block_sum(sq);
        if (__builtin_amdgcn_workitem_id_x() == 0) o.partials[w] = bs;
    }
}

template <typename T, int EPI, int TZB>
__global__ __launch_bounds__(256, sizeof(acc_t<T>) != 4 ? 2 : 6) void k_backward(BwdOut<T>, GeoDev g, const T *__restrict__ proj,
                                                                                const int *__restrict__ skip, int nbx,
                                                                                int nby, int nbz)
{
    if (skip && *skip) return;
    constexpr int CHC = ch_cols(TZB);
    __shared__ PixStage<acc_t<T>, split_records<acc_t<T>>(TZB)> s_pix[(ch_rows(TZB) + 1) * CHC + NH - 1];
    __shared__ ColStage s_col[CHC];
    __shared__ float s_row[ch_rows(TZB) + 1];
    backward_block<T, EPI, TZB, CHC>(g, __builtin_amdgcn_workgroup_id_x(), proj, nbx, nby, nbz, s_pix, s_col, s_row,
                                     [] { return late_out<T>(); });
}

static BwdPlan brick_plan(const GeoDev &g, int form)
{
    BwdPlan p{};
    p.form = form;
    p.tz = form == BWD_DEEP ? TZ_DEEP : TZ;
    p.sets = 1;
    p.nbx = (g.nx + BX - 1) / BX;
    p.nby = (g.ny + BY - 1) / BY;
    p.nbz = (g.nz + p.tz - 1) / p.tz;
    p.nblocks = (int64_t)p.nbx * p.nby * p.nbz;
    return p;
}

// Expected shadow of n voxel columns a side and tz layers, in pixels at the
// isocentre's magnification: columns over the diagonal, rows (of the layers that the
// volume has), each with a little for the nearer half of the orbit and for the ends.
static float shadow_cols(const GeoDev &g, int n)
{
    return 1.05f * 1.4142f * (float)n * fmaxf(g.vx, g.vy) * g.ku / g.sid + 2.0f;
}
static float shadow_rows(const GeoDev &g, int tz)
{
    return 1.1f * (float)(tz < g.nz ? tz : g.nz) * g.vz * g.kv / g.sid + 3.0f;
}

// View subsets of the wave form, at most `most` (a power of two): none without a view
// but in the last octave, and for fewer than eight views the number of the least
// ceil(views / subsets) x wavefronts, a chip of 4096 wavefronts counting as full; one and two
// subsets cost 10 and 5 % more per view.  Measured (us, 4 / 2 / 1 subsets; n, q as
// below): n 192, q 1.25, 1 view 78.5 / - / 25.1, 2 views - / 33.9 / 37.4, 4 views 51.0 / 53.9 / 62.1,
// 6 views 82.1 / 76.7 / 90.2; n 256, q 2.2, 1 view 191 / - / 81, 3 views 266 / 218 / 201; n 400,
// q 1.25, 4 views 404 / 394 / 389; 2048^2 x 4, q 0.7, 30 views 841 / 870 / 882.
int wave_sets(int64_t bricks, int most, int views)
{
    int sets = most;
    while (sets / 2 >= views) sets /= 2;
    if (views >= 8) return sets;
    float best = INFINITY;
    int chosen = sets;
    for (int s = sets; s >= 1; s /= 2) {
        const int64_t waves = bricks * s < 4096 ? 4096 : bricks * s;
        const float cost = (float)((views + s - 1) / s) * (float)waves * (s == 1 ? 1.1f : (s == 2 ? 1.05f : 1.0f));
        if (cost < best) {
            best = cost;
            chosen = s;
        }
    }
    return chosen;
}

// Bricks and view subsets that one launch can hold (a grid has less than 2^32
// threads): fewer subsets, then deeper bricks, for the flattest of the largest volumes.
void wave_fit_launch(const GeoDev &g, BwdPlan &p)
{
    for (;;) {
        p.nbz = (g.nz + p.tz - 1) / p.tz;
        p.nblocks = (int64_t)p.nbx * p.nby * p.nbz;
        if (p.nblocks * 64 * p.sets < (int64_t)1 << 32) return;
        if (p.sets > 1) p.sets /= 2;
        else p.tz *= 2;
    }
}

// Wave form: the deepest brick whose shadow is expected to fit one chunk (or nearly so:
// a second chunk now and then costs less than shallower bricks) and that leaves enough
// bricks, and as many view subsets as fill the chip.  Measured (us, cube of n voxels, q
// detector pixels per voxel at the isocentre, depth 32 / 16 / 8 / 4):
// n 128, q 0.7: 287 / 338 / 413 / -; n 192, q 1.25: 2179 / 1129 / 1487 / 1984;
// n 192, q 1.6: 4288 / 1673 / 1729 / 2235; n 256, q 1.6: 24322 / 9777 / 10485 / 14020;
// n 192, q 2.2: - / 4389 / 2929 / 3364; n 192, q 3.2: - / 12665 / 8635 / 7236; n 64, q 1.6:
// - / 118 / 81 / 94.  4 or 8 subsets: 2048 bricks (n 128, q 1.25) 668 / 543, 4096 (n 128,
// q 2.2) 1444 / 1373, 6912 (n 192, q 1.25) 1175 / 1129, 16384 (n 256, q 1) 5685 / 5735, 31250
// (n 400, q 1.25) 4759 / 4876.  No deeper than the volume: 1024^2 x 6, q 2.2, 8 views in
// double precision, 8- / 4-deep 249 / 347.
// For few views more bricks, as many wavefronts as eight views give (n 96, q 1.25, 1 view, 16- / 8- /
// 4-deep 11.4 / 8.9 / 8.4).
static BwdPlan wave_plan(const GeoDev &g, bool single)
{
    BwdPlan p{};
    p.form = BWD_WAVES;
    p.nbx = (g.nx + WX - 1) / WX;
    p.nby = (g.ny + WY - 1) / WY;
    const float cols = shadow_cols(g, WX);
    const int few = 1536 / (g.nviews < 8 ? g.nviews : 8);
    for (p.tz = 32; p.tz > 4; p.tz /= 2) {
        if (p.tz / 2 >= g.nz) continue;
        const float records = cols * (shadow_rows(g, p.tz) + 1.0f);
        p.nbz = (g.nz + p.tz - 1) / p.tz;
        if (p.tz == 32 && 7 * g.nz < 5 * 32 * p.nbz) continue;  // all 32 layers are taken (layer_test)
        p.nblocks = (int64_t)p.nbx * p.nby * p.nbz;
        const float over = p.tz == 8 ? 1.3f : (p.tz == 16 && single ? 1.1f : 1.0f);
        if (records <= over * (float)wave_cap(single && split_records<float>(p.tz)) && p.nblocks >= (p.tz == 32 && few < 1024 ? 1024 : few))
            break;
    }
    p.nbz = (g.nz + p.tz - 1) / p.tz;
    p.nblocks = (int64_t)p.nbx * p.nby * p.nbz;
    // (bricks of 32: one subset per wavefront of the batched form, whose second set of
    // sums would not fit its registers)
    const int most = p.tz == 32 || p.nblocks > (single ? 8192 : 2048) ? 4 : (p.nblocks > 512 ? 8 : 16);
    p.sets = wave_sets(p.nblocks, most, g.nviews);
    wave_fit_launch(g, p);
    return p;
}

// A single backprojection's form (single: with single-precision accumulation).  Deep
// workgroup bricks where there are enough of them to fill the chip and their shadow
// is expected to fit one staged chunk; 16-deep ones where the same holds and the
// volume is so large that the wave form's own staging of every 8 x 8 columns costs more
// than the workgroup's barriers; wave form elsewhere.
// Measured (us, wave form / 16-deep / 32-deep bricks; n and q as above, n 256 with 90
// views at q 0.7 and 300 elsewhere):
//   q 0.7:  n 192 657 / 788 / 694, n 256 1100 / 1013 / 982, n 400 2826 / 2429 / 1835
//   q 1:    n 256 5686 / 5955 / 7188, n 400 3884 / 3898 / 3817
//   q 1.25: n 192 1129 / 1555 / 2276, n 256 6627 / 6882 / 12587, n 400 4759 / 4602 / 6751
//   q 1.6:  n 256 9777 / 10723 / -, n 320 3679 / 3806 / -, n 400 7145 / 6823 / 12867
//   q 2.2:  n 256 17924 / 27169 / -, n 400 12890 / 17528 / -
// With fewer than eight views the wavefronts of a workgroup brick all work on each of
// them, and the 16-deep bricks pay from 300 bricks per view on (wave form / 16-deep): q 1.25,
// n 192 (1728 bricks) 1 view 25.1 / 19.8, 2 views 33.9 / 31.5, 4 views 51.7 / 55.2, 6 views 76.7 / 82.1;
// n 256 (4096 bricks) 1 view 44.0 / 32.0, 6 views 160 / 143, 8 views 196 / 184, 20 views 454 / 456;
// 256^2 x 68 (1280 bricks) 4 views 36.1 / 32.7, 30 views 199 / 219; 311 x 305 x 228 with voxels 1.4 as
// high (6000 bricks) 2 views 100 / 91, 4 views 169 / 169, 8 views 288 / 324, 20 views 664 / 793.
// Double precision takes the deep bricks for volumes of 128 layers and more only: 16- /
// 32-deep 512^2 x 40, q 0.7, 30 views 280 / 347, 1024^2 x 1, 60 views 372 / 464; n 256, 30 views
// 373 / 352.
static BwdPlan plan(const GeoDev &g, bool deep_allowed, bool single = true)
{
    const BwdPlan deep = brick_plan(g, BWD_DEEP), shallow = brick_plan(g, BWD_BRICKS);
    const float cols = shadow_cols(g, BX);
    if (deep_allowed && (single || g.nz >= 128) && deep.nblocks >= 2048 && cols <= (float)ch_cols(TZ_DEEP) &&
        shadow_rows(g, TZ_DEEP) <= (float)ch_rows(TZ_DEEP))
        return deep;
    const int enough = single ? 12288 : 4096, per_view = 300;
    if (shallow.nblocks >= (g.nviews < 8 ? per_view * g.nviews : enough) && cols <= (float)ch_cols(TZ) &&
        shadow_rows(g, TZ) <= (float)ch_rows(TZ))
        return shallow;
    return wave_plan(g, single);
}

BwdPlan backward_plan(const GeoDev &g, bool single) { return plan(g, true, single); }

BwdPlan backward_plan_variant(const GeoDev &g, int variant)
{
    return variant == BWD_VDEEP ? brick_plan(g, BWD_DEEP) : plan(g, false);
}

// The variant a single solve would use: its block decomposition (and so its
// partial sums) is that of kct_cgls_solve.
int backward_default_variant(const GeoDev &g) { return backward_plan(g).form == BWD_DEEP ? BWD_VDEEP : BWD_VSHALLOW; }

// LDS of a workgroup brick in the batched form: records, columns, row factors.
constexpr size_t brick_lds_bytes(int tz)
{
    const size_t rec = split_records<float>(tz) ? sizeof(PixStage<float, true>) : sizeof(PixStage<float, false>);
    return ((ch_rows(tz) + 1) * ch_cols(tz) + NH - 1) * rec + ch_cols(tz) * sizeof(ColStage) + (ch_rows(tz) + 1) * sizeof(float);
}
constexpr size_t lds_max(size_t a, size_t b) { return a > b ? a : b; }
constexpr size_t batch_lds_bytes(bool deep)
{
    return deep ? lds_max(wave_lds_bytes<float, false>(W_GROUPS), brick_lds_bytes(TZ_DEEP))
                : lds_max(wave_lds_bytes<float, true>(W_GROUPS), brick_lds_bytes(TZ));
}

// Instance bi's BwdOut (read at once: reading it late keeps bi alive and cost the batched
// kernels more, 8 uneven instances 44.0 -> 49.7 ms).
__device__ __forceinline__ auto batch_out(const BatchInst *bi)
{
    return [o = BwdOut<float>{bi->r, nullptr, bi->sc, bi->part, nullptr}] { return o; };
}

template <int TZB>
__device__ __forceinline__ void batch_brick(const BatchInst *bi, const BwdPlan &p, int lw, char *lds)
{
    using Rec = PixStage<float, split_records<float>(TZB)>;
    Rec *s_pix = reinterpret_cast<Rec *>(lds);
    ColStage *s_col = reinterpret_cast<ColStage *>(s_pix + (ch_rows(TZB) + 1) * ch_cols(TZB) + NH - 1);
    float *s_row = reinterpret_cast<float *>(s_col + ch_cols(TZB));
    backward_block<float, BWD_NORM, TZB, ch_cols(TZB)>(bi->g, lw, bi->e, p.nbx, p.nby, p.nbz, s_pix, s_col, s_row,
                                                       batch_out(bi));
}

// One tile (brick) of instance bi's r = A^T e with |r|^2 partials.  Wave form: the
// four wavefronts take the view subsets of the single solve in turns.
// DEEP: an instance whose bricks are 32 voxels deep, else one of the other forms.
template <bool DEEP>
__device__ __forceinline__ void batch_backward_tile(const BatchInst *bi, int lw, char *lds)
{
    const BwdPlan p = bi->bwd;
    const auto out = batch_out(bi);
    if constexpr (DEEP) {
        if (p.form == BWD_DEEP)
            batch_brick<TZ_DEEP>(bi, p, lw, lds);
        else
            backward_wave_block<float, BWD_NORM, 32, true>(bi->g, lw, bi->e, p.nbx, p.nby, p.nbz, W_GROUPS, p.sets, lds, out);
        return;
    }
    if (p.form == BWD_BRICKS) batch_brick<TZ>(bi, p, lw, lds);
    else if (p.tz == 16)
        backward_wave_block<float, BWD_NORM, 16, true>(bi->g, lw, bi->e, p.nbx, p.nby, p.nbz, W_GROUPS, p.sets, lds, out);
    else if (p.tz == 8)
        backward_wave_block<float, BWD_NORM, 8, true>(bi->g, lw, bi->e, p.nbx, p.nby, p.nbz, W_GROUPS, p.sets, lds, out);
    else
        backward_wave_block<float, BWD_NORM, 4, true>(bi->g, lw, bi->e, p.nbx, p.nby, p.nbz, W_GROUPS, p.sets, lds, out);
}

// Persistent batched r = A^T e: every workgroup takes items from the queue
// until it is empty (see BatchInst); each item is up to BATCH_ITEM_BWD bricks
// of one instance.  Two kernels, each with the instances of its forms: the 32-deep
// bricks' sums need 96 registers and their records 31 KiB of LDS, the others' 80 and
// 26, so the others run six workgroups per compute unit instead of five.
template <bool DEEP>
__global__ __launch_bounds__(256, DEEP ? 5 : 6) void kp_backward(const BatchInst *__restrict__ B,
                                                      const int64_t *__restrict__ off, int count,
                                                      BatchQueue *__restrict__ q)
{
    __shared__ __align__(16) char lds[batch_lds_bytes(DEEP)];
    const int64_t total = off[count];
    unsigned passed = 0;
    for (;;) {
        const int64_t item = batch_pop(q, total, passed);
        if (item >= total) break;
        const int i = batch_find(off, count, item);
        const BatchInst *bi = B + i;
        if (bi->sc->done) continue;
        const int64_t t0 = (item - off[i]) * BATCH_ITEM_BWD;
        const int64_t t1 = t0 + BATCH_ITEM_BWD < bi->nbk ? t0 + BATCH_ITEM_BWD : bi->nbk;
        for (int64_t t = t0; t < t1; ++t) {
            batch_backward_tile<DEEP>(bi, (int)t, lds);
            __syncthreads();  // the tile's block sum is read before the next tile writes it
        }
    }
    batch_exit(q);
}

hipError_t batch_backward_occupancy(int &per_cu, int &per_cu_deep)
{
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kp_backward<false>, 256, 0);
    return e != hipSuccess ? e : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_deep, kp_backward<true>, 256, 0);
}

// off and off_deep: the items of the instances of either kernel; q[0] and q[1] their queues.  A
// kernel without instances (grid 0) is not launched.
hipError_t launch_batch_backward(const BatchInst *B, const int64_t *off, const int64_t *off_deep, int count, BatchQueue *q,
                                 int grid, int grid_deep, hipStream_t st)
{
    if (grid_deep > 0)
        hipLaunchKernelGGL(kp_backward<true>, dim3((unsigned)grid_deep), dim3(256), 0, st, B, off_deep, count, q + 1);
    if (grid > 0) hipLaunchKernelGGL(kp_backward<false>, dim3((unsigned)grid), dim3(256), 0, st, B, off, count, q);
    return hipGetLastError();
}

template <typename T, int EPI>
static void launch_bricks(const GeoDev &g, const BwdPlan &p, const T *proj, T *out, T *out_z, const Scalars *sc,
                          double *partials, const int *skip, const float *aux, hipStream_t st)
{
    const dim3 grid((unsigned)p.nblocks);
    const BwdOut<T> o{out, out_z, sc, partials, aux};
    if (p.form == BWD_DEEP)
        hipLaunchKernelGGL((k_backward<T, EPI, TZ_DEEP>), grid, dim3(256), 0, st, o, g, proj, skip, p.nbx, p.nby, p.nbz);
    else
        hipLaunchKernelGGL((k_backward<T, EPI, TZ>), grid, dim3(256), 0, st, o, g, proj, skip, p.nbx, p.nby, p.nbz);
}

// A single plain backprojection with batched-form variant v (the tuner times these).
hipError_t launch_backward_variant(const GeoDev &g, int variant, const float *proj, float *out, hipStream_t st)
{
    const BwdPlan p = backward_plan_variant(g, variant);
    if (p.form == BWD_WAVES)
        return launch_backward_waves<float>(g, p, proj, out, nullptr, BWD_PLAIN, nullptr, nullptr, nullptr, st, nullptr);
    launch_bricks<float, BWD_PLAIN>(g, p, proj, out, nullptr, nullptr, nullptr, nullptr, nullptr, st);
    return hipGetLastError();
}

// Workgroups (and partial sums) of a single backprojection with g.
int64_t backward_num_blocks(const GeoDev &g)
{
    return (g.projector == KCT_PROJECTOR_TT ? tt_backward_plan(g) : backward_plan(g)).nblocks;
}

template <typename T>
hipError_t launch_backward(const GeoDev &g, const T *proj, T *out, T *out_z, int epi, const Scalars *sc,
                           double *partials, const int *skip, hipStream_t st, const float *aux)
{
    if (g.projector == KCT_PROJECTOR_TT) return launch_backward_tt<T>(g, proj, out, out_z, epi, sc, partials, skip, st, aux);
    const BwdPlan p = backward_plan(g, !std::is_same<T, double>::value);
    if (p.form == BWD_WAVES) return launch_backward_waves<T>(g, p, proj, out, out_z, epi, sc, partials, skip, st, aux);
    if constexpr (std::is_same<T, double>::value) {  // double storage: plain backprojection only
        if (epi != BWD_PLAIN) return hipErrorInvalidValue;
        launch_bricks<T, BWD_PLAIN>(g, p, proj, out, out_z, sc, partials, skip, aux, st);
    } else {
        switch (epi) {
        case BWD_PLAIN: launch_bricks<T, BWD_PLAIN>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_NORM: launch_bricks<T, BWD_NORM>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_LSQR0: launch_bricks<T, BWD_LSQR0>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_LSQR: launch_bricks<T, BWD_LSQR>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_TIK: launch_bricks<T, BWD_TIK>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_JACOBI: launch_bricks<T, BWD_JACOBI>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        default:
            if constexpr (std::is_same<T, float>::value) {  // the diagonal of A^T A is single precision
                if (epi == BWD_DIAG) {
                    launch_bricks<T, BWD_DIAG>(g, p, proj, out, out_z, sc, partials, skip, aux, st);
                    break;
                }
                if (epi == BWD_DIAG_INV) {
                    launch_bricks<T, BWD_DIAG_INV>(g, p, proj, out, out_z, sc, partials, skip, aux, st);
                    break;
                }
            }
            return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

#define KCT_BINST(T)                                                                                             \
    template hipError_t launch_backward<T>(const GeoDev &, const T *, T *, T *, int, const Scalars *, double *, \
                                           const int *, hipStream_t, const float *);
KCT_BINST(float)
KCT_BINST(bf16)
KCT_BINST(_Float16)
KCT_BINST(double)

}  // namespace kct
