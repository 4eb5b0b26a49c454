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
    int *arrivals;        // ARRIVAL_WORDS, for route_finish
    int *counts;          // batches with a finishing workgroup: tallied by it (zeroed beforehand)
    int64_t N;
    int K, D;
    float *cnorm_out, *cinit_out;   // small batches: where a launch that computes the norms itself leaves them
    int retained_only;
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
// call asks for it.  What the others leave behind are atomics alone, so a workgroup only waits for its own to
// be done before it reports; a release fence would write back, and its acquire half invalidate, the XCD's L2
// once per workgroup.  Reports go to ARRIVAL_FAN words first and from there to one: atomics on one word take
// turns at about 13 ns.
// `smem`: sizeof(PlanLdsSmall) bytes of LDS, free by now, when the call asks for the grouping.
template <int NT>
__device__ __forceinline__ void route_finish(const RouteKParams &p, char *smem)
{
    __shared__ int last_flag;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned n = gridDim.x, f = blockIdx.x % ARRIVAL_FAN;
        bool last = true;
        if (n > ARRIVAL_FAN) {
            const unsigned mine = (n - f + ARRIVAL_FAN - 1) / ARRIVAL_FAN;   // workgroups that report to word f
            last = atomicAdd(p.arrivals + (1 + f) * ARRIVAL_STRIDE, 1) == (int)mine - 1;
        }
        if (last) last = atomicAdd(p.arrivals, 1) == (int)min(n, (unsigned)ARRIVAL_FAN) - 1;
        last_flag = last;
    }
    __syncthreads();
    if (!last_flag) return;
    if (p.self_clean && p.counts) {   // (uniform) nobody zeroed the histogram ahead of this launch
        for (int k = threadIdx.x; k < p.K; k += NT) p.counts[k] = 0;
        __syncthreads();
    }
    if (p.self_clean && threadIdx.x <= ARRIVAL_FAN) p.arrivals[threadIdx.x * ARRIVAL_STRIDE] = 0;
    // The grouping's own inputs: the offsets on their way beside the winners, the experts handed over in LDS.
    constexpr bool MAY_PLAN = NT == PLAN_THREADS_SMALL;
    PlanLdsSmall &L = *reinterpret_cast<PlanLdsSmall *>(smem);
    constexpr int OFFS = PLAN_CAP_SMALL / PLAN_THREADS_SMALL + 1;
    int off[OFFS];
    if constexpr (MAY_PLAN) {
        if (p.with_plan) {
#pragma unroll
            for (int u = 0; u < OFFS; ++u) off[u] = p.seq_offsets[min((int)threadIdx.x + u * NT, (int)p.N)];
        }
    }
    constexpr int UNR = 4;   // the loads of several queries in flight: each is a trip to memory
    for (int q0 = threadIdx.x; q0 < (int)p.N; q0 += NT * UNR) {
        int bi[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int q = min(q0 + u * NT, (int)p.N - 1);
            const unsigned idx =
                (unsigned)(__hip_atomic_load(&p.best[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xffffffffu);
            bi[u] = (idx < (unsigned)p.K) ? (int)idx : 0;   // nothing won: centroid 0
        }
        int e[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) e[u] = p.slot ? p.slot[bi[u]] : bi[u];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int q = q0 + u * NT;
            if (q >= (int)p.N) break;
            if (p.cid) p.cid[q] = bi[u];
            if (p.expert_ids) p.expert_ids[q] = e[u];
            if constexpr (MAY_PLAN)
                if (p.with_plan) L.ekey[q] = (unsigned)e[u];   // (at most PLAN_CAP_SMALL queries)
            if (p.counts) atomicAdd(&p.counts[bi[u]], 1);
        }
    }
    if (p.self_clean) {   // ready for the next call (every thread its own queries, read above; lanes past the end read the last)
        lds_barrier();
        for (int q = threadIdx.x; q < (int)p.N; q += NT) p.best[q] = ~0ull;
    }
    if constexpr (MAY_PLAN) {
        if (p.with_plan) {
#pragma unroll
            for (int u = 0; u < OFFS; ++u)
                if ((int)threadIdx.x + u * NT <= (int)p.N) L.off[threadIdx.x + u * NT] = off[u];
            plan_body<PLAN_THREADS_SMALL, PLAN_CAP_SMALL, true>(p.plan, nullptr, nullptr, p.rank_of_expert, p.err_word, L);
        }
    }
}

}  // namespace moin
