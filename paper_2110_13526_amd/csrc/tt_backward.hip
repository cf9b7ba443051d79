// tt_backward.hip -- the TT footprint projector's transpose, r = A^T e (kct_tt.h), with
// single-precision accumulation, in the wave form of the Siddon pair's (kct_wave.h): one
// wavefront per brick of WX x WY voxel columns and view subset stages the brick's
// detector shadow as L_i e_i in its own LDS region; each lane takes the detector
// columns of its voxel column's transaxial footprint and, per voxel, the rows of
// its axial footprint.  Neighbouring voxels share the ramp of the plane between them.
// Bounded by VALU issue.  With bricks of 16 x 16 x 16 voxels per workgroup, a trapezoid per
// voxel and branches in its integral, 128^3 x 180 views, 154 x 120 detector took 2.92 ms (512
// workgroups); this form 1.02 ms. 512^3 x 720, 616 x 480: 330 -> 216 ms.
#include <type_traits>

#include "kct_epilogue.h"
#include "kct_internal.h"
#include "kct_tt.h"
#include "kct_wave.h"
#include "kct_weights.h"

namespace kct {

// Staged values of a chunk.  512 / 768 / 1024 (us; cube of n voxels, q detector pixels per
// voxel): n 192, q 2.2, 30 views 1227 / 1055 / 1057; n 96, q 4, 20 views 482 / 384 / 309; n 128, q 0.7, 60
// views 311 / 308 / 309; n 400, q 0.7, 20 views 2670 / 2646 / 2655; else within 0.5 %.
constexpr int TTB_CAP = 768;
constexpr int TTB_COLS = 48;   // most columns of a chunk
constexpr int TTB_NC = 4;      // detector columns at once
static_assert(TTB_CAP >= W_SUMS * 64, "the partial sums fit a staging region");

constexpr size_t ttb_lds_bytes(int waves) { return (size_t)waves * (TTB_CAP * sizeof(float) + sizeof(double)); }

// The deepest brick whose shadow is expected to fit one chunk (see TTB_CAP), and view
// subsets by the number of bricks, four from 2048 bricks on (the Siddon pair's wave form: from
// 8192): with the limit at 8192, n 192 (3456 bricks) q 0.7, 60 views 1000 against 901 us, q
// 1.25, 30 views 784 / 666, q 2.2, 30 views 1061 / 1055; n 256 and 128 the same.
BwdPlan tt_backward_plan(const GeoDev &g)
{
    BwdPlan p{};
    p.form = BWD_WAVES;
    p.nbx = (g.nx + WX - 1) / WX;
    p.nby = (g.ny + WY - 1) / WY;
    const float cols = 1.05f * 1.4142f * (float)WX * fmaxf(g.vx, g.vy) * g.ku / g.sid + 3.0f;
    const int few = 1536 / (g.nviews < 8 ? g.nviews : 8);
    for (p.tz = 16;; p.tz /= 2) {
        if (p.tz > 4 && p.tz / 2 >= g.nz) continue;  // (no deeper than the volume)
        p.nbz = (g.nz + p.tz - 1) / p.tz;
        p.nblocks = (int64_t)p.nbx * p.nby * p.nbz;
        const float rows = 1.1f * (float)(p.tz < g.nz ? p.tz : g.nz) * g.vz * g.kv / g.sid + 3.0f;
        if (p.tz == 4 || (cols * rows <= (float)TTB_CAP && p.nblocks >= few)) break;
    }
    p.sets = wave_sets(p.nblocks, p.nblocks > 2048 ? 4 : (p.nblocks > 512 ? 8 : 16), g.nviews);
    wave_fit_launch(g, p);
    return p;
}

template <typename T, int EPI, int TZB, bool OVERLAP>
__global__ __launch_bounds__(1024, 5) void k_backward_tt(GeoDev g, const T *__restrict__ proj, T *__restrict__ out,
                                                         T *__restrict__ out_z, const Scalars *__restrict__ sc,
                                                         double *__restrict__ partials, const int *__restrict__ skip,
                                                         int nbx, int nby, int nbz, const float *__restrict__ aux)
{
    extern __shared__ __align__(16) char lds[];
    if (skip && *skip) return;
    constexpr bool SQ = EPI == BWD_DIAG || EPI == BWD_DIAG_INV;  // squared weights, e not read
    const int waves = (int)(__builtin_amdgcn_workgroup_size_x() >> 6);
    const int wave = __builtin_amdgcn_readfirstlane((int)(__builtin_amdgcn_workitem_id_x() >> 6));
    const int lane = (int)(__builtin_amdgcn_workitem_id_x() & 63);
    float *s_all = reinterpret_cast<float *>(lds), *s_le = s_all + wave * TTB_CAP;
    double *red = reinterpret_cast<double *>(s_all + waves * TTB_CAP);

    // XCD-aware brick assignment (see backproject.hip)
    constexpr int XCDS = 8;
    const int nb = nbx * nby * nbz, w = (int)__builtin_amdgcn_workgroup_id_x();
    const int b = (nb % XCDS == 0) ? (w % XCDS) * (nb / XCDS) + w / XCDS : w;
    const int bx = b % nbx, by = (b / nbx) % nby, bz = b / (nbx * nby);
    const int ix = bx * WX + lane % WX, iy = by * WY + lane / WX;
    const int iz0 = bz * TZB;
    const int nzb = g.nz - iz0 < TZB ? g.nz - iz0 : TZB;
    const bool valid = ix < g.nx && iy < g.ny;
    const int cnx = g.nx - bx * WX < WX ? g.nx - bx * WX : WX, cny = g.ny - by * WY < WY ? g.ny - by * WY : WY;
    const float ex = 0.5f * (float)cnx * g.vx, ey = 0.5f * (float)cny * g.vy;
    const float xc = g.x0 + (float)(bx * WX) * g.vx + ex, yc = g.y0 + (float)(by * WY) * g.vy + ey;
    const float wz0 = g.z0 + (float)iz0 * g.vz, wz1 = g.z0 + (float)(iz0 + nzb) * g.vz;

    float acc[TZB];
#pragma unroll
    for (int j = 0; j < TZB; ++j) acc[j] = 0.0f;

    for (int k = wave; k < g.nviews; k += waves) {
        const ViewParam vp = g.views[k];
        // shadow of the brick: pixels whose extent (centre +- 0.5) meets the bounds of its
        // corners' images (see kct_wave.h), 0.01 pixel more against rounding
        int u0, u1, v0, v1;
        {
            const float dn = __builtin_fmaf(ex, fabsf(vp.s), ey * fabsf(vp.c));
            const float dd = __builtin_fmaf(ex, fabsf(vp.c), ey * fabsf(vp.s));
            const float dx = xc - vp.sx, dy = yc - vp.sy;
            const float num = __builtin_fmaf(vp.c, dy, -vp.s * dx);
            const float den = __builtin_fmaf(-vp.c, dx, -vp.s * dy);
            const float inv = rcp_approx(den), rmax = rcp_approx(den - dd), rmin = rcp_approx(den + dd);
            const float fc = __builtin_fmaf(num * inv, g.ku, g.fu0);
            const float hc = __builtin_fmaf(__builtin_fmaf(dd * fabsf(num), inv, dn) * rmax, g.ku, 0.51f);
            const float p0 = wz0 * rmin, p1 = wz0 * rmax, p2 = wz1 * rmin, p3 = wz1 * rmax;
            const float zlo = fminf(fminf(p0, p1), fminf(p2, p3)), zhi = fmaxf(fmaxf(p0, p1), fmaxf(p2, p3));
            const int c0 = (int)ceilf(fc - hc), c1 = (int)floorf(fc + hc);
            const int r0 = (int)ceilf(__builtin_fmaf(zlo, g.kv, g.fv0) - 0.51f);
            const int r1 = (int)floorf(__builtin_fmaf(zhi, g.kv, g.fv0) + 0.51f);
            u0 = __builtin_amdgcn_readfirstlane(c0 < 0 ? 0 : c0);
            u1 = __builtin_amdgcn_readfirstlane(c1 > g.nu - 1 ? g.nu - 1 : c1);
            v0 = __builtin_amdgcn_readfirstlane(r0 < 0 ? 0 : r0);
            v1 = __builtin_amdgcn_readfirstlane(r1 > g.nv - 1 ? g.nv - 1 : r1);
        }
        const T *pk = SQ ? proj : proj + (size_t)k * g.nv * g.nu;  // not read when SQ
        const ColParam *ck = g.cols + (size_t)k * g.nu;
        TTTrap tu{};
        float ka = 0.0f, kb = 0.0f;
        if (valid) {
            float dmin, dmax, rdmin, rdmax;
            tt_transaxial(g, vp, ix, iy, tu, dmin, dmax, rdmin, rdmax);
            tt_row_scales(g, rdmin, rdmax, ka, kb);
        }
        constexpr int RMAX = TTB_CAP / 8;  // rows that leave room for 8 columns
        for (int cv0 = v0; cv0 <= v1; cv0 += RMAX) {
            const int nrow = v1 - cv0 + 1 < RMAX ? v1 - cv0 + 1 : RMAX;
            int cmax = TTB_COLS;
            if (nrow * cmax > TTB_CAP) {
                // TTB_CAP / nrow through a reciprocal, one less where that rounds up
                cmax = __builtin_amdgcn_readfirstlane((int)((float)TTB_CAP * __builtin_amdgcn_rcpf((float)nrow) + 0.01f));
                if (nrow * cmax > TTB_CAP) --cmax;
            }
            for (int cu0 = u0; cu0 <= u1; cu0 += cmax) {
                const int ncol = u1 - cu0 + 1 < cmax ? u1 - cu0 + 1 : cmax;
                // stage L e, a fixed column per lane (see kct_wave.h)
                {
                    const float rn = __builtin_amdgcn_rcpf((float)ncol);
                    const int step = __builtin_amdgcn_readfirstlane((int)(64.5f * rn));
                    const int r0 = (int)(((float)lane + 0.5f) * rn), c = lane - r0 * ncol;
                    if (r0 < step) {
                        const ColParam cp = *byte_at<ColParam>(ck, (unsigned)(cu0 + c) * (unsigned)sizeof(ColParam));
                        unsigned pix = ((unsigned)(cv0 + r0) * (unsigned)g.nu + (unsigned)(cu0 + c)) * (unsigned)sizeof(T);
                        unsigned row = (unsigned)(cv0 + r0) * (unsigned)sizeof(RowParam);
                        float *to = s_le + (r0 * ncol + c);
                        for (int r = r0; r < nrow; r += step) {
                            const float ev = SQ ? 0.0f : to_f32(*byte_at<T>(pk, pix));
                            const RowParam rp = *byte_at<RowParam>(g.rows, row);
                            const float amp = tt_amplitude(ray_length_per_xi(cp.lxy2, rp.qz, cp.gp), cp.inv_a,
                                                           zeta_inv_slope(rp.inv_qz, cp.kz));
                            *to = SQ ? amp * amp : amp * ev;
                            pix += (unsigned)(step * g.nu) * (unsigned)sizeof(T);
                            row += (unsigned)step * (unsigned)sizeof(RowParam);
                            to += step * ncol;
                        }
                    }
                }
                wave_lds_order();
                if (valid)
                    tt_gather_ramps<float, SQ, OVERLAP, TTB_NC, TZB>(g, iz0, tu.t, ka, kb, s_le, ncol, cu0, ncol, cv0, nrow, nzb, acc);
                wave_lds_order();
            }
        }
    }

    // every voxel's partial sums through LDS, in order within a group of subsets, then the groups
    double sq = 0.0;
    const int per = waves > W_GROUPS ? waves / W_GROUPS : 1;
#pragma unroll
    for (int j0 = 0; j0 < TZB; j0 += W_SUMS) {
        if (j0 > 0) __syncthreads();
#pragma unroll
        for (int j = j0; j < j0 + W_SUMS && j < TZB; ++j) s_le[(j - j0) * 64 + lane] = acc[j];
        __syncthreads();
        const int jend = nzb < j0 + W_SUMS ? nzb : j0 + W_SUMS;
        for (int j = j0 + wave; j < jend; j += waves) {
            const int at = (j - j0) * 64 + lane;
            float v[W_GROUPS];
#pragma unroll
            for (int q = 0; q < W_GROUPS; ++q) {
                v[q] = 0.0f;
                if (q * per >= waves) continue;
                v[q] = s_all[q * per * TTB_CAP + at];
                for (int i = 1; i < per; ++i) v[q] += s_all[(q * per + i) * TTB_CAP + at];
            }
            if (valid) {
                const int iz = iz0 + j;
                const size_t vox = ((size_t)iz * g.ny + iy) * g.nx + ix;
                sq += bwd_store<T, EPI, float>(out, out_z, sc, aux, vox, ((size_t)iy * g.nx + ix) * g.nz + iz,
                                               (v[0] + v[1]) + (v[2] + v[3]));
            }
        }
    }
    if (bwd_has_partials<EPI>()) {
        for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
        if (lane == 0) red[wave] = sq;
        __syncthreads();
        if (__builtin_amdgcn_workitem_id_x() == 0) {
            double r = red[0];
            for (int q = 1; q < waves; ++q) r += red[q];
            partials[w] = r;
        }
    }
}

template <typename T, int EPI, bool OVERLAP>
static void launch_btt_depth(const GeoDev &g, const BwdPlan &p, const T *proj, T *out, T *out_z, const Scalars *sc,
                             double *partials, const int *skip, const float *aux, hipStream_t st)
{
    const dim3 grid((unsigned)p.nblocks), block(64u * (unsigned)p.sets);
    const unsigned lds = (unsigned)ttb_lds_bytes(p.sets);
    if (p.tz == 16)
        hipLaunchKernelGGL((k_backward_tt<T, EPI, 16, OVERLAP>), grid, block, lds, st, g, proj, out, out_z, sc, partials,
                           skip, p.nbx, p.nby, p.nbz, aux);
    else if (p.tz == 8)
        hipLaunchKernelGGL((k_backward_tt<T, EPI, 8, OVERLAP>), grid, block, lds, st, g, proj, out, out_z, sc, partials,
                           skip, p.nbx, p.nby, p.nbz, aux);
    else
        hipLaunchKernelGGL((k_backward_tt<T, EPI, 4, OVERLAP>), grid, block, lds, st, g, proj, out, out_z, sc, partials,
                           skip, p.nbx, p.nby, p.nbz, aux);
}

template <typename T, int EPI>
static void launch_btt(const GeoDev &g, const T *proj, T *out, T *out_z, const Scalars *sc, double *partials,
                       const int *skip, const float *aux, hipStream_t st)
{
    const BwdPlan p = tt_backward_plan(g);
    if (g.tt_overlap) launch_btt_depth<T, EPI, true>(g, p, proj, out, out_z, sc, partials, skip, aux, st);
    else launch_btt_depth<T, EPI, false>(g, p, proj, out, out_z, sc, partials, skip, aux, st);
}

template <typename T>
hipError_t launch_backward_tt(const GeoDev &g, const T *proj, T *out, T *out_z, int epi, const Scalars *sc,
                              double *partials, const int *skip, hipStream_t st, const float *aux)
{
    if constexpr (std::is_same<T, double>::value) {
        return launch_backward_tt_f64(g, proj, out, epi, skip, st);
    } else {
        switch (epi) {
        case BWD_PLAIN: launch_btt<T, BWD_PLAIN>(g, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_NORM: launch_btt<T, BWD_NORM>(g, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_LSQR0: launch_btt<T, BWD_LSQR0>(g, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_LSQR: launch_btt<T, BWD_LSQR>(g, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_TIK: launch_btt<T, BWD_TIK>(g, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_JACOBI: launch_btt<T, BWD_JACOBI>(g, proj, out, out_z, sc, partials, skip, aux, st); break;
        default:
            if constexpr (std::is_same<T, float>::value) {
                if (epi == BWD_DIAG) {
                    launch_btt<T, BWD_DIAG>(g, proj, out, out_z, sc, partials, skip, aux, st);
                    break;
                }
                if (epi == BWD_DIAG_INV) {
                    launch_btt<T, BWD_DIAG_INV>(g, proj, out, out_z, sc, partials, skip, aux, st);
                    break;
                }
            }
            return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

#define KCT_TTB(T)                                                                                                \
    template hipError_t launch_backward_tt<T>(const GeoDev &, const T *, T *, T *, int, const Scalars *, double *, \
                                              const int *, hipStream_t, const float *);
KCT_TTB(float)
KCT_TTB(bf16)
KCT_TTB(_Float16)
KCT_TTB(double)

}  // namespace kct
