// Grouping of a batch by expert: sequences are sorted by (expert id, sequence
// index) and cut into row tiles that never span two sequences, so every tile
// has exactly one adapter (Section 1: one expert per query; Section 4.1: id -1
// = no adapter, base model only).  For small batches and short sequences the tokens
// themselves are grouped by expert instead, so that the decode kernels read each distinct
// adapter once.  Everything happens on the device in one workgroup: the host
// never looks at the ids.  Offsets that do not tile [0, T) in order make the
// whole batch base-only (and raise the sticky fault): every output row is still
// written.
#include "kernels.h"
#include "plan_body.h"

namespace moin {

template <int PT, int CAP>
__global__ __launch_bounds__(PT) void plan_kernel(PlanView pv, const int *seq_offsets, const int *expert_ids,
                                                  const int *rank_of_expert, int *err_word)
{
    extern __shared__ __align__(16) char smem[];
    plan_body<PT, CAP>(pv, seq_offsets, expert_ids, rank_of_expert, err_word,
                       *reinterpret_cast<PlanLds<PT, CAP> *>(smem));
}

// Batches of more sequences than LDS holds: a bitonic sort through the plan's global scratch.
constexpr int PLAN_LDS_S = 2048;

// In-place exclusive prefix sum of data[0..n) by one workgroup; returns the total.
template <int PLAN_THREADS>
__device__ int block_exclusive_scan(int *data, int n, int *lds /* PLAN_THREADS + 1 ints */)
{
    const int tid = threadIdx.x;
    const int per = (n + PLAN_THREADS - 1) / PLAN_THREADS;
    const int lo = min(tid * per, n), hi = min(lo + per, n);
    int sum = 0;
    for (int i = lo; i < hi; ++i) sum += data[i];
    lds[tid] = sum;
    __syncthreads();
    // Hillis-Steele inclusive scan over the per-thread sums
    for (int off = 1; off < PLAN_THREADS; off <<= 1) {
        const int v = (tid >= off) ? lds[tid - off] : 0;
        __syncthreads();
        lds[tid] += v;
        __syncthreads();
    }
    const int total = lds[PLAN_THREADS - 1];
    int run = lds[tid] - sum;
    __syncthreads();
    for (int i = lo; i < hi; ++i) {
        const int v = data[i];
        data[i] = run;
        run += v;
    }
    __syncthreads();
    return total;
}

__global__ __launch_bounds__(PLAN_THREADS_MAX) void plan_large_kernel(PlanView pv, const int *seq_offsets,
                                                                      const int *expert_ids,
                                                                      const int *rank_of_expert, int *err_word)
{
    constexpr int PLAN_THREADS = PLAN_THREADS_MAX;
    __shared__ int lds[PLAN_THREADS + 1];
    __shared__ unsigned long long lds_keys[PLAN_LDS_S];
    __shared__ int bad_offsets;
    const int tid = threadIdx.x;
    const int S = pv.S;
    const int T = (int)pv.T;
    int npow2 = 1;
    while (npow2 < S) npow2 <<= 1;
    unsigned long long *keys = pv.keys;
    int *tmp = pv.tmp;

    int *lens = tmp;                  // [S]   length of each sequence (by sequence)
    int *a1 = tmp + (S + 1);          // [S+1] per sorted position: tile count -> tile base
    int *a2 = tmp + 2 * (S + 1);      // [S+1] per sorted position: length -> token base
    int *a3 = tmp + 3 * (S + 1);      // [S+1] per sorted position: group head flag -> group id

    // 1. validate, build sort keys (expert + 1 in the high word: -1 sorts first)
    int err = 0;
    if (tid == 0) bad_offsets = 0;
    __syncthreads();
    if (tid == 0 && (seq_offsets[0] != 0 || seq_offsets[S] != T)) err |= ERR_BAD_OFFSETS;
    for (int s = tid; s < npow2; s += PLAN_THREADS) {
        unsigned long long key = ~0ull;
        if (s < S) {
            int lo = seq_offsets[s], hi = seq_offsets[s + 1];
            int e = expert_ids[s];
            if (lo < 0 || hi > T || hi < lo) {
                err |= ERR_BAD_OFFSETS;
                lo = 0;
                hi = 0;
            }
            if (e < -1 || e >= pv.E) {
                err |= ERR_BAD_EXPERT;
                e = -1;
            }
            if (plan_rank_of(e, rank_of_expert, err_word) == 0) e = -1;   // rank 0: base model only
            lens[s] = hi - lo;
            key = ((unsigned long long)(unsigned)(e + 1) << 32) | (unsigned)s;
        }
        keys[s] = key;
    }
    if (err) atomicOr(err_word, err);
    if (err & ERR_BAD_OFFSETS) bad_offsets = 1;
    plan_plain_tiles(pv, PLAN_THREADS);
    __syncthreads();
    if (bad_offsets) {
        plan_base_only(pv, PLAN_THREADS);
        return;
    }

    // 2. bitonic sort of the keys by the one workgroup.  Element i meets element i ^ j,
    // ascending where (i & k) == 0.  Only the steps whose partners lie PLAN_LDS_S or more apart walk global
    // memory; all steps with j < PLAN_LDS_S stay inside an aligned chunk of PLAN_LDS_S
    // keys, which is brought into LDS once for a whole run of them.
    auto steps_in = [&](unsigned long long *buf, int n, int base, int k, int j_first) {
        for (int j = j_first; j > 0; j >>= 1) {
            for (int i = tid; i < n; i += PLAN_THREADS) {
                const int l = i ^ j;
                if (l > i) {
                    const unsigned long long a = buf[i], b = buf[l];
                    const bool up = ((base + i) & k) == 0;
                    if ((a > b) == up) {
                        buf[i] = b;
                        buf[l] = a;
                    }
                }
            }
            __syncthreads();
        }
    };
    auto chunk_run = [&](int c, int k_first, int k_last, int j_first_of_last) {
        // chunk c through LDS: whole stages k_first..k_last / 2 and, of stage k_last, the steps from j_first_of_last down
        unsigned long long *g = keys + (size_t)c * PLAN_LDS_S;
        for (int i = tid; i < PLAN_LDS_S; i += PLAN_THREADS) lds_keys[i] = g[i];
        __syncthreads();
        for (int k = k_first; k < k_last; k <<= 1) steps_in(lds_keys, PLAN_LDS_S, c * PLAN_LDS_S, k, k >> 1);
        steps_in(lds_keys, PLAN_LDS_S, c * PLAN_LDS_S, k_last, j_first_of_last);
        for (int i = tid; i < PLAN_LDS_S; i += PLAN_THREADS) g[i] = lds_keys[i];
        __syncthreads();
    };
    const int n_chunks = npow2 / PLAN_LDS_S;
    for (int c = 0; c < n_chunks; ++c) chunk_run(c, 2, PLAN_LDS_S, PLAN_LDS_S >> 1);
    for (int k = 2 * PLAN_LDS_S; k <= npow2; k <<= 1) {
        for (int j = k >> 1; j >= PLAN_LDS_S; j >>= 1) {
            for (int i = tid; i < npow2; i += PLAN_THREADS) {
                const int l = i ^ j;
                if (l > i) {
                    const unsigned long long a = keys[i], b = keys[l];
                    const bool up = (i & k) == 0;
                    if ((a > b) == up) {
                        keys[i] = b;
                        keys[l] = a;
                    }
                }
            }
            __syncthreads();
        }
        for (int c = 0; c < n_chunks; ++c) chunk_run(c, k, k, PLAN_LDS_S >> 1);
    }

    // 3. per sorted position: tile count, token count, group-head flag
    for (int p = tid; p < S; p += PLAN_THREADS) {
        const unsigned long long key = keys[p];
        const int s = (int)(key & 0xffffffffu);
        const int len = lens[s];
        a1[p] = (len + TILE_M - 1) / TILE_M;
        a2[p] = len;
        const bool head = (p == 0) || ((keys[p - 1] >> 32) != (key >> 32));
        a3[p] = head ? 1 : 0;
    }
    __syncthreads();
    const int n_tiles = block_exclusive_scan<PLAN_THREADS>(a1, S, lds);
    if (tid == 0) *pv.n_tiles = min(n_tiles, pv.max_tiles);
    int n_groups = 0, n_tok = 0;
    if (pv.decode) {
        n_tok = block_exclusive_scan<PLAN_THREADS>(a2, S, lds);
        n_groups = block_exclusive_scan<PLAN_THREADS>(a3, S, lds);   // a3[p] = groups before p
        if (tid == 0) pv.grp_start[n_groups] = min(n_tok, T);
    }

    // 4. emit
    for (int p = tid; p < S; p += PLAN_THREADS) {
        const unsigned long long key = keys[p];
        const int s = (int)(key & 0xffffffffu);
        const int e = (int)(key >> 32) - 1;
        const int lo = seq_offsets[s];
        const int len = lens[s];
        const int tb = a1[p];
        const int rk = plan_rank_of(e, rank_of_expert, err_word);
        for (int j = 0, left = len; left > 0 && tb + j < pv.max_tiles; ++j, left -= TILE_M) {
            pv.tile_row0[tb + j] = lo + j * TILE_M;
            pv.tile_rows[tb + j] = min(left, TILE_M);
            pv.tile_expert[tb + j] = e;
            pv.tile_rank[tb + j] = rk;
        }
        if (pv.decode) {
            const int base = min(a2[p], T);
            const bool head = (p == 0) || ((keys[p - 1] >> 32) != (key >> 32));
            if (head) {
                const int gi = a3[p];   // exclusive count of heads before p
                pv.grp_tmp[gi] = make_int2(e, rk);
                pv.grp_start[gi] = base;
            }
        }
    }
    if (pv.decode) {
        // tokens in sorted order, one per thread and step whatever the sequences' lengths:
        // position t belongs to the last sorted sequence that starts at or before it
        for (int t = tid; t < min(n_tok, T); t += PLAN_THREADS) {
            int first = 0, last = S - 1;
            while (first < last) {
                const int mid = (first + last + 1) >> 1;
                if (a2[mid] <= t) first = mid;
                else last = mid - 1;
            }
            const int s = (int)(keys[first] & 0xffffffffu);
            pv.tok_sorted[t] = seq_offsets[s] + (t - a2[first]);
        }
    }
    if (pv.decode) {
        // A group ends where the next one starts.  It is cut into records of at most
        // pv.chunk tokens: the decode kernels hand a record to one column of
        // workgroups, and a hot expert's tokens must not all queue behind one column.
        __syncthreads();   // grp_start / grp_tmp are complete, a1 is free
        for (int gi = tid; gi < n_groups; gi += PLAN_THREADS)
            a1[gi] = (pv.grp_start[gi + 1] - pv.grp_start[gi] + pv.chunk - 1) / pv.chunk;
        __syncthreads();
        const int n_rec = min(block_exclusive_scan<PLAN_THREADS>(a1, n_groups, lds), pv.max_groups);
        for (int gi = tid; gi < n_groups; gi += PLAN_THREADS) {
            const int2 er = pv.grp_tmp[gi];
            const int ge = pv.grp_start[gi + 1];
            int rec = a1[gi];
            for (int t = pv.grp_start[gi]; t < ge && rec < pv.max_groups; t += pv.chunk, ++rec)
                pv.grp_meta[rec] = make_int4(er.x, t, min(t + pv.chunk, ge), er.y);
        }
        if (tid == 0) {
            pv.n_groups[0] = n_rec;
            // (base-only sequences sort first; a1 holds the records before each group)
            pv.n_groups[1] = pv.grp_tmp[0].x >= 0 ? 0 : n_groups > 1 ? min(a1[1], pv.max_groups) : n_rec;
        }
        // unused records read as empty groups, so the decode kernels need not
        // fetch the group count before their own record
        for (int gi = n_rec + tid; gi < pv.max_groups; gi += PLAN_THREADS) pv.grp_meta[gi] = make_int4(-1, 0, 0, 0);
    }
}

hipError_t prepare_plan_kernels()
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&plan_kernel<PLAN_THREADS_MAX, PLAN_CAP_MAX>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(PlanLdsMax));
}

hipError_t launch_plan(const PlanView &pv, const int *seq_offsets, const int *expert_ids,
                       const int *rank_of_expert, int *err_word, hipStream_t stream)
{
    if (pv.S <= PLAN_CAP_SMALL)
        hipLaunchKernelGGL((plan_kernel<PLAN_THREADS_SMALL, PLAN_CAP_SMALL>), dim3(1), dim3(PLAN_THREADS_SMALL),
                           sizeof(PlanLdsSmall), stream, pv, seq_offsets, expert_ids, rank_of_expert, err_word);
    else if (pv.S <= PLAN_CAP_MAX)
        hipLaunchKernelGGL((plan_kernel<PLAN_THREADS_MAX, PLAN_CAP_MAX>), dim3(1), dim3(PLAN_THREADS_MAX),
                           sizeof(PlanLdsMax), stream, pv, seq_offsets, expert_ids, rank_of_expert, err_word);
    else
        hipLaunchKernelGGL(plan_large_kernel, dim3(1), dim3(PLAN_THREADS_MAX), 0, stream, pv, seq_offsets,
                           expert_ids, rank_of_expert, err_word);
    return hipGetLastError();
}

}  // namespace moin
