// backproject_wave.hip -- launches of the backprojection's wave form (kct_wave.h):
// r = A^T e (Section 2, Eq. 2) for volumes that have too few 16 x 16 column bricks
// to fill the chip, and for shadows too wide for those bricks' staged chunk.
#include <type_traits>

#include "kct_internal.h"
#include "kct_wave.h"

namespace kct {

// Waves per SIMD that the LDS of the staging regions leaves room for: 6 with split
// records, 5 with whole ones.
template <typename T, int EPI, int TZB>
__global__ __launch_bounds__(1024, sizeof(acc_t<T>) != 4 ? 2 : (TZB < TZ_DEEP ? 6 : 5)) void k_backward_waves(
    BwdOut<T>, GeoDev g, const T *__restrict__ proj, const int *__restrict__ skip, int nbx, int nby, int nbz)
{
    extern __shared__ __align__(16) char lds[];
    if (skip && *skip) return;
    const int waves = (int)(__builtin_amdgcn_workgroup_size_x() >> 6);
    backward_wave_block<T, EPI, TZB, false>(g, __builtin_amdgcn_workgroup_id_x(), proj, nbx, nby, nbz, waves, waves, lds,
                                            [] { return late_out<T>(); });
}

template <typename T, int EPI>
static void launch_waves(const GeoDev &g, const BwdPlan &p, const T *proj, T *out, T *out_z, const Scalars *sc,
                         double *partials, const int *skip, const float *aux, hipStream_t st)
{
    const dim3 grid((unsigned)p.nblocks), block(64u * (unsigned)p.sets);
    using A = acc_t<T>;
    const BwdOut<T> o{out, out_z, sc, partials, aux};
    const unsigned lds = (unsigned)(split_records<A>(p.tz) ? wave_lds_bytes<A, true>(p.sets) : wave_lds_bytes<A, false>(p.sets));
    switch (p.tz) {
    case 32:
        hipLaunchKernelGGL((k_backward_waves<T, EPI, 32>), grid, block, lds, st, o, g, proj, skip, p.nbx, p.nby,
                           p.nbz);
        break;
    case 16:
        hipLaunchKernelGGL((k_backward_waves<T, EPI, 16>), grid, block, lds, st, o, g, proj, skip, p.nbx, p.nby,
                           p.nbz);
        break;
    case 8:
        hipLaunchKernelGGL((k_backward_waves<T, EPI, 8>), grid, block, lds, st, o, g, proj, skip, p.nbx, p.nby,
                           p.nbz);
        break;
    default:
        hipLaunchKernelGGL((k_backward_waves<T, EPI, 4>), grid, block, lds, st, o, g, proj, skip, p.nbx, p.nby,
                           p.nbz);
    }
}

template <typename T>
hipError_t launch_backward_waves(const GeoDev &g, const BwdPlan &p, const T *proj, T *out, T *out_z, int epi,
                                 const Scalars *sc, double *partials, const int *skip, hipStream_t st,
                                 const float *aux)
{
    if constexpr (std::is_same<T, double>::value) {  // double storage: plain backprojection only
        if (epi != BWD_PLAIN) return hipErrorInvalidValue;
        launch_waves<T, BWD_PLAIN>(g, p, proj, out, out_z, sc, partials, skip, aux, st);
    } else {
        switch (epi) {
        case BWD_PLAIN: launch_waves<T, BWD_PLAIN>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_NORM: launch_waves<T, BWD_NORM>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_LSQR0: launch_waves<T, BWD_LSQR0>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_LSQR: launch_waves<T, BWD_LSQR>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_TIK: launch_waves<T, BWD_TIK>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        case BWD_JACOBI: launch_waves<T, BWD_JACOBI>(g, p, proj, out, out_z, sc, partials, skip, aux, st); break;
        default:
            if constexpr (std::is_same<T, float>::value) {  // the diagonal of A^T A is single precision
                if (epi == BWD_DIAG) {
                    launch_waves<T, BWD_DIAG>(g, p, proj, out, out_z, sc, partials, skip, aux, st);
                    break;
                }
                if (epi == BWD_DIAG_INV) {
                    launch_waves<T, BWD_DIAG_INV>(g, p, proj, out, out_z, sc, partials, skip, aux, st);
                    break;
                }
            }
            return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

#define KCT_WINST(T)                                                                                              \
    template hipError_t launch_backward_waves<T>(const GeoDev &, const BwdPlan &, const T *, T *, T *, int,        \
                                                 const Scalars *, double *, const int *, hipStream_t, const float *);
KCT_WINST(float)
KCT_WINST(bf16)
KCT_WINST(_Float16)
KCT_WINST(double)

}  // namespace kct
