// kct_batch.h -- device helpers of the batched kernels.
#pragma once

#include "kct_internal.h"

namespace kct {

// The instance that owns workgroup w of a batched grid: the largest i with
// off[i] <= w (off is ascending, count + 1 entries, off[0] = 0).
__device__ __forceinline__ int batch_find(const int64_t *__restrict__ off, int count, int64_t w)
{
    int lo = 0, hi = count;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= w) lo = mid;
        else hi = mid;
    }
    // the same instance in every lane (w is the workgroup's): keep the
    // instance's fields in scalar registers
    return __builtin_amdgcn_readfirstlane(lo);
}

// The next of a persistent step's `total` items, the same in every thread of the
// workgroup; total when none is left.  The items are dealt to one queue per XCD (item
// modulo BATCH_XCDS; the resident workgroups of the step fill the XCDs in turn), so
// that tiles which share projections or volume columns run on the XCD whose L2 holds
// them, as they do in a separate solve's launch; a workgroup whose queue is empty draws
// from the next one's.  Each queue hands out its items in increasing order and every
// workgroup draws until all are empty, so the queues always drain.  passed (0 at first,
// thread 0's): the queues that this workgroup has found empty; an empty one stays so
// for the launch and is not asked again.  The others' counters are read before one is
// drawn from, all at once: a draw from an empty queue by every workgroup of every
// XCD is what a small batch spent its time on (2 x 24^3, 12 views: 766 us per iteration with
// eight draws each, 411 with one queue, 258 in this form and with no more workgroups
// than items).
__device__ __forceinline__ int64_t batch_pop(BatchQueue *q, int64_t total, unsigned &passed)
{
    __shared__ unsigned s_item;
    __syncthreads();  // the previous item's readers are done with s_item
    if (__builtin_amdgcn_workitem_id_x() == 0) {
        unsigned item = (unsigned)total, first = __builtin_amdgcn_workgroup_id_x();
        unsigned seen[BATCH_XCDS];
        while (passed < BATCH_XCDS) {
            const unsigned c = (first + passed) % BATCH_XCDS;
            const unsigned drawn = atomicAdd(&q->next[c].n, 1u) * BATCH_XCDS + c;
            if (drawn < (unsigned)total) {
                item = drawn;
                break;
            }
            // the next one that is not empty yet
#pragma unroll
            for (unsigned s = 1; s < BATCH_XCDS; ++s)
                seen[s] = __hip_atomic_load(&q->next[(first + s) % BATCH_XCDS].n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned at = BATCH_XCDS;
#pragma unroll
            for (unsigned s = BATCH_XCDS - 1; s >= 1; --s)
                if (s > passed && seen[s] * BATCH_XCDS + (first + s) % BATCH_XCDS < (unsigned)total) at = s;
            passed = at;
        }
        s_item = item;
    }
    __syncthreads();
    return (int64_t)s_item;
}

// Leave a persistent step: the last workgroup to leave (every other one has
// drawn its final item) resets the queues for the next launch of the step.
__device__ __forceinline__ void batch_exit(BatchQueue *q)
{
    if (__builtin_amdgcn_workitem_id_x() == 0) {
        __threadfence();
        const unsigned n = atomicAdd(&q->exited, 1u);
        if (n == __builtin_amdgcn_grid_size_x() / __builtin_amdgcn_workgroup_size_x() - 1) {
            for (unsigned c = 0; c < BATCH_XCDS; ++c) atomicExch(&q->next[c].n, 0u);
            atomicExch(&q->exited, 0u);
        }
    }
}

}  // namespace kct
