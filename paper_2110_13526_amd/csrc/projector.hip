// projector.hip -- the forward projector's rules and launches (the kernels are in
// kct_forward.h, the backprojector in backproject.hip), and its persistent batched
// form.
#include <type_traits>

#include "kct_batch.h"
#include "kct_forward.h"
#include "kct_internal.h"

namespace kct {

// Rows per lane: a wavefront's time goes with 7 + 5.5 R (its in-plane walk and each
// row's part), so R is the one with the least bands x that; a detector of few rows
// leaves lanes without a ray otherwise.  Measured (us, R 1 / 2 / 3 / 4): 96 rows (64^3 x 90)
// 93 / 70 / - / 131; 120 rows (128^3 x 720) 1419 / 955 / - / 1498; 218 rows (96^3 x 186)
// 757 / 477 / 534 / 385; 384 rows (256^3 x 360) 11775 / 7304 / 5523 / 5991; 480 rows
// (512^3 x 720, ms) 93.9 / 64.2 / 62.5 / 60.7.
// Divided walks where the columns of all views give fewer than five wavefronts
// per SIMD (one or two rows per lane): 576 wavefronts (16^3 x 12) 21.4 -> 19.4 us, 840
// (24^3 x 40) 26.6 -> 20.2, 4860 (64^3 x 90, 48 rows) 52 -> 43; 6391 (45 x 37 x 51 x 77)
// 41 -> 49, 8640 (64^3 x 90, 96 rows) 70 -> 74.
FwdPlan forward_plan(const GeoDev &g)
{
    FwdPlan p{1, false};
    float best = 0.0f;
    for (int r = 1; r <= 4; ++r) {
        const float cost = (float)fwd_grid(g, r).nbands * (7.0f + 5.5f * (float)r);
        if (r == 1 || cost < best) {
            best = cost;
            p.rows = r;
        }
    }
    return forward_plan_rows(g, p.rows);
}

// The plan with a given number of rows per lane (the batched form's tuner sets it).
FwdPlan forward_plan_rows(const GeoDev &g, int rows)
{
    return FwdPlan{rows, rows <= 2 && fwd_grid(g, rows).nblocks * FWD_COLS <= 5120};
}

// Whether a plain projection reads the volume in its own layout although it has room
// for the z-fastest copy: a divided walk of a volume of up to 32^3 voxels, which the
// L1 and L2 hold, takes less longer than the copy's launch costs.  Measured (us, with
// the copy / in place): 16^3 x 12 views 11.7 / 8.7; 24^3 x 60 11.3 / 8.8; 32^3 x 60 15.0 /
// 12.3; but 32^3 x 200 (not divided) 32 / 39, 40^3 x 60 17.5 / 19.7, 48^3 x 60 22 / 32.
bool forward_in_place(const GeoDev &g)
{
    return g.projector == KCT_PROJECTOR_SIDDON && (int64_t)g.nx * g.ny * g.nz <= 32768 && forward_plan(g).divided;
}

int64_t forward_num_blocks(const GeoDev &g)
{
    return g.projector == KCT_PROJECTOR_TT ? tt_forward_num_blocks(g) : fwd_grid(g, forward_plan(g).rows).nblocks;
}
int64_t forward_num_blocks_r(const GeoDev &g, int rows_per_lane) { return fwd_grid(g, rows_per_lane).nblocks; }

template <typename TV, typename TP>
static hipError_t launch_forward_plan(const GeoDev &g, FwdPlan p, const TV *vol, const TV *vol_z, TP *out, const TP *aux,
                                      int epi, const Scalars *sc, double *partials, const int *skip, hipStream_t st)
{
    switch (p.rows) {
    case 1: return launch_forward_rows<TV, TP, 1>(g, p.divided, vol, vol_z, out, aux, epi, sc, partials, skip, st);
    case 2: return launch_forward_rows<TV, TP, 2>(g, p.divided, vol, vol_z, out, aux, epi, sc, partials, skip, st);
    case 3: return launch_forward_rows<TV, TP, 3>(g, p.divided, vol, vol_z, out, aux, epi, sc, partials, skip, st);
    case 4: return launch_forward_rows<TV, TP, 4>(g, p.divided, vol, vol_z, out, aux, epi, sc, partials, skip, st);
    default: return hipErrorInvalidValue;
    }
}

template <typename TV, typename TP>
hipError_t launch_forward(const GeoDev &g, const TV *vol, const TV *vol_z, TP *out, const TP *aux, int epi,
                          const Scalars *sc, double *partials, const int *skip, hipStream_t st)
{
    if (g.projector == KCT_PROJECTOR_TT) return launch_forward_tt<TV, TP>(g, vol, vol_z, out, aux, epi, sc, partials, skip, st);
    return launch_forward_plan<TV, TP>(g, forward_plan(g), vol, vol_z, out, aux, epi, sc, partials, skip, st);
}

hipError_t launch_forward_r(const GeoDev &g, const float *vol, const float *vol_z, float *out, int rows_per_lane,
                            hipStream_t st)
{
    return launch_forward_plan<float, float>(g, forward_plan_rows(g, rows_per_lane), vol, vol_z, out, nullptr, FWD_PLAIN, nullptr, nullptr, nullptr, st);
}

// One tile (workgroup) of instance bi's p = A d with |p|^2 partials, in its rows per
// lane; walks that its own solve divides among wavefronts are taken share by share.
template <int R, int WALK> __device__ __forceinline__ void batch_forward_rows(const BatchInst *bi, int64_t t)
{
    forward_block<float, float, FWD_NORM, R, WALK, true>(bi->g, t, nullptr, bi->dz, bi->p, nullptr, bi->sc, bi->part,
                                                         nullptr);
}
__device__ __forceinline__ void batch_forward_tile(const BatchInst *bi, int64_t t)
{
    const FwdPlan p = bi->fwd;
    if (p.rows == 1) {
        if (p.divided) batch_forward_rows<1, FWD_IN_TURN>(bi, t);
        else batch_forward_rows<1, FWD_WHOLE>(bi, t);
    } else if (p.rows == 2) {
        if (p.divided) batch_forward_rows<2, FWD_IN_TURN>(bi, t);
        else batch_forward_rows<2, FWD_WHOLE>(bi, t);
    } else if (p.rows == 3) {
        batch_forward_rows<3, FWD_WHOLE>(bi, t);
    } else {
        batch_forward_rows<4, FWD_WHOLE>(bi, t);
    }
}

// Persistent batched p = A d with |p|^2 partials for every instance (CGLS
// steps of a batched solve): every workgroup takes items from the queue until
// it is empty; an item is up to BATCH_ITEM_FWD workgroup tiles of one
// instance's forward grid, in its own rows-per-lane variant.
__global__ __launch_bounds__(256, 7) void kp_forward(const BatchInst *__restrict__ B, const int64_t *__restrict__ off,
                                                  int count, BatchQueue *__restrict__ q)
{
    const int64_t total = off[count];
    unsigned passed = 0;
    for (;;) {
        const int64_t item = batch_pop(q, total, passed);
        if (item >= total) break;
        const int i = batch_find(off, count, item);
        const BatchInst *bi = B + i;
        if (bi->sc->done) continue;
        // Eight consecutive items take the tiles of one run in turn, so that an item's tiles
        // are all those of one XCD in the forward's own order; the last items, which do
        // not fill such a run, take consecutive tiles.
        constexpr int64_t RUN = (int64_t)BATCH_ITEM_FWD * BATCH_XCDS;
        const int64_t m = item - off[i], run = m / BATCH_XCDS * RUN;
        const bool whole = run + RUN <= bi->nf;
        const int64_t step = whole ? BATCH_XCDS : 1, t0 = whole ? run + m % BATCH_XCDS : m * BATCH_ITEM_FWD;
        const int64_t tend = t0 + step * BATCH_ITEM_FWD, t1 = tend < bi->nf ? tend : bi->nf;
        for (int64_t t = t0; t < t1; t += step) {
            batch_forward_tile(bi, t);
            __syncthreads();  // the tile's block sum is read before the next tile writes it
        }
    }
    batch_exit(q);
}

hipError_t launch_batch_forward(const BatchInst *B, const int64_t *off, int count, BatchQueue *q, int grid,
                                hipStream_t st)
{
    hipLaunchKernelGGL(kp_forward, dim3((unsigned)grid), dim3(256), 0, st, B, off, count, q);
    return hipGetLastError();
}

// Resident workgroups of the persistent batched kernels: the device's compute
// units times the workgroups one of them holds.
hipError_t batch_persistent_grids(int &fwd, int &bwd, int &bwd_deep, int &dir)
{
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    int nf = 0, nb = 0, nbd = 0, nd = 0;
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nf, kp_forward, 256, 0);
    if (e == hipSuccess) e = batch_backward_occupancy(nb, nbd);
    if (e == hipSuccess) e = batch_dir_occupancy(nd);
    if (e != hipSuccess) return e;
    fwd = cus * (nf > 0 ? nf : 1);
    bwd = cus * (nb > 0 ? nb : 1);
    bwd_deep = cus * (nbd > 0 ? nbd : 1);
    dir = cus * (nd > 0 ? nd : 1);
    return hipSuccess;
}

#define KCT_INST(TV, TP)                                                                                       \
    template hipError_t launch_forward<TV, TP>(const GeoDev &, const TV *, const TV *, TP *, const TP *, int,   \
                                               const Scalars *, double *, const int *, hipStream_t);
KCT_INST(float, float)
KCT_INST(bf16, bf16)
KCT_INST(_Float16, _Float16)
KCT_INST(float, bf16)
KCT_INST(float, _Float16)
KCT_INST(double, double)

}  // namespace kct
