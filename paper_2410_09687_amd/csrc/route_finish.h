// What the routing kernels that split the centroid range over workgroups share: their parameters, and the
// end of a launch in which the last workgroup turns the packed per-query minima into ids.
#pragma once
#include "gemm_core.h"
#include "kernels.h"
#include "plan_body.h"

namespace moin {

struct RouteKParams {
    const char *emb, *cent;
    const float *cnorm;   // [K padded to a multiple of 256]; +inf for excluded / padding
    const float *cinit;   // [same]: -||c||^2 / 2, -inf for excluded / padding
    const int *slot;
    int *cid;
    int *expert_ids;
    unsigned long long *best;
    int *arrivals;        // for route_finish
    int *counts;          // batches with a finishing workgroup: tallied by it (zeroed beforehand)
    int64_t N;
    int K, D;
    int group;            // streaming kernel: workgroups that share one query tile
    int64_t n_virtual;    // streaming kernel: work items (query tiles rounded up to 8, times group)
    int finish;           // the workgroup that arrives last turns best[] into ids (route_finish)
    int self_clean;       // finishing kernels: best / arrivals are clean on entry and are left clean
                          // (the finishing workgroup resets them and zeroes counts before its tally)
    // optional: the finishing workgroup goes on to group the routed batch by
    // expert (queries = the batch's sequences), so that routing and grouping are one launch
    int with_plan;
    PlanView plan;
    const int *seq_offsets, *rank_of_expert;
    int *err_word;
};

// Every workgroup of the launch calls this once its winners are in best[] (device-scope atomics).  The one
// that arrives last unpacks them: ids, adapter slots, the histogram, and the grouping of the batch where the
// call asks for it.
template <int NT>
__device__ __forceinline__ void route_finish(const RouteKParams &p)
{
    __shared__ int last_flag;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0)
        last_flag = (atomicAdd(p.arrivals, 1) == (int)gridDim.x - 1);
    __syncthreads();
    if (!last_flag) return;
    __threadfence();
    if (p.self_clean && p.counts) {   // (uniform) nobody zeroed the histogram ahead of this launch
        for (int k = threadIdx.x; k < p.K; k += NT) p.counts[k] = 0;
        __syncthreads();
    }
    if (p.self_clean && threadIdx.x == 0) *p.arrivals = 0;
    for (int q = threadIdx.x; q < (int)p.N; q += NT) {
        const unsigned long long key =
            __hip_atomic_load(&p.best[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (p.self_clean) p.best[q] = ~0ull;   // ready for the next call
        const unsigned idx = (unsigned)(key & 0xffffffffu);
        const int bi = (idx < (unsigned)p.K) ? (int)idx : 0;   // nothing won: centroid 0
        if (p.cid) p.cid[q] = bi;
        if (p.expert_ids) p.expert_ids[q] = p.slot ? p.slot[bi] : bi;
        if (p.counts) atomicAdd(&p.counts[bi], 1);
    }
    if constexpr (NT == PLAN_THREADS_SMALL) {
        if (p.with_plan) {
            // the ids this workgroup has just written are the plan's input
            __threadfence_block();
            __syncthreads();
            plan_body<PLAN_THREADS_SMALL>(p.plan, p.seq_offsets, p.expert_ids, p.rank_of_expert, p.err_word);
        }
    }
}

}  // namespace moin
