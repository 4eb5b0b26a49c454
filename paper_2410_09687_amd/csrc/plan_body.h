// Grouping of a batch by expert, as device functions (see plan.hip for what they compute).
#pragma once
#include "gemm_core.h"
#include "kernels.h"

namespace moin {

constexpr int PLAN_THREADS_MAX = 1024;   // large batches
constexpr int PLAN_THREADS_SMALL = 256;  // up to PLAN_CAP_SMALL sequences: four waves meet at a barrier much faster than sixteen
constexpr int PLAN_CAP_SMALL = 512;
constexpr int PLAN_CAP_MAX = 12288;      // what one compute unit's LDS holds, at 12 bytes a sequence
// Up to here a sequence's place is found by comparing it with all others (200 sequences: 7.8 us, a radix sort 6.6).
constexpr int PLAN_COUNT_S = 128;

// (The arrays are always reached through the struct, never through a pointer that could also be a global one: for
// such a generic pointer the compiler may form &array[-1] ahead of a loop, and below the start of LDS that is an
// address outside every segment.)
template <int PT, int CAP>
struct PlanLds {
    static constexpr bool KEEPS = CAP <= PLAN_CAP_SMALL;
    alignas(KEEPS ? 16 : 4) unsigned ekey[CAP];   // expert + 1 of each sequence (-1, no adapter, sorts first)
    int tokbase[CAP];            // per sorted position: tokens before it
    uint16_t idx[2][CAP];        // sequences in sorted order, and the buffer they are sorted through
    int hist[PT / 64][128];      // per wave: digit counts, then cursors
    int sums[3][PT / 64];
    int bad_offsets, any_long;
    // What every sequence has in memory, where there is room for it: read once, on the way in.  (At the end: two words ahead of
    // the other arrays cost the large kernel 0.6 us of 8.4.)
    int off[KEEPS ? CAP + 1 : 1];     // sequence offsets
    int rank[KEEPS ? CAP : 1];        // of the sequence's adapter
};
using PlanLdsSmall = PlanLds<PLAN_THREADS_SMALL, PLAN_CAP_SMALL>;
using PlanLdsMax = PlanLds<PLAN_THREADS_MAX, PLAN_CAP_MAX>;

// Barrier for what goes through LDS.  Nothing written to memory is read back, so four waves wait for LDS alone (__syncthreads also
// waits until every store has arrived); sixteen waves are faster by __syncthreads (1024 sequences: 10.9 us for the kernel, 11.5).
template <int PT>
__device__ __forceinline__ void plan_meet()
{
    if constexpr (PT == PLAN_THREADS_SMALL) lds_barrier();
    else __syncthreads();
}

// Exclusive prefix sums of N values per thread over the workgroup, and the totals.
template <int PT, int N>
__device__ __forceinline__ void plan_scan(int (&v)[N], int (&total)[N], int (*sums)[PT / 64])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int own[N];
#pragma unroll
    for (int k = 0; k < N; ++k) own[k] = v[k];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int y = __shfl_up(v[k], off);
            if (lane >= off) v[k] += y;
        }
    if (lane == 63)
#pragma unroll
        for (int k = 0; k < N; ++k) sums[k][wave] = v[k];
    plan_meet<PT>();
#pragma unroll
    for (int k = 0; k < N; ++k) {
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < PT / 64; ++w) {
            const int s = sums[k][w];
            before += w < wave ? s : 0;
            all += s;
        }
        v[k] += before - own[k];
        total[k] = all;
    }
    plan_meet<PT>();
}

// Rank of adapter slot e ("Future Works": adaptive rank per topic).  Multiples of 8,
// like the stacks' own rank; anything else is rounded down and raises the sticky fault.
__device__ __forceinline__ int plan_rank_of(int e, const int *rank_of_expert, int *err_word)
{
    if (e < 0) return 0;
    if (!rank_of_expert) return RANK_FULL;
    int rk = rank_of_expert[e];
    if (rk < 0 || (rk & 7)) {
        atomicOr(err_word, ERR_BAD_RANK);
        rk = rk < 0 ? RANK_FULL : (rk & ~7);
    }
    return rk;
}

// Plain row tiles over all tokens (batches of the gather path).
__device__ __forceinline__ void plan_plain_tiles(const PlanView &pv, int nt)
{
    const int T = (int)pv.T;
    for (int j = threadIdx.x; j < pv.max_plain; j += nt) {
        pv.plain_row0[j] = j * TILE_M;
        pv.plain_rows[j] = max(min(TILE_M, T - j * TILE_M), 0);
        pv.plain_expert[j] = -1;
        pv.plain_rank[j] = 0;
    }
    if (threadIdx.x == 0 && pv.max_plain > 0) *pv.plain_n = min(pv.max_plain, (T + TILE_M - 1) / TILE_M);
}

// The sequences do not cover every token exactly once: one base-only sequence over the whole batch instead.
__device__ __forceinline__ void plan_base_only(const PlanView &pv, int nt_threads)
{
    const int tid = threadIdx.x, T = (int)pv.T;
    const int nt = (T + TILE_M - 1) / TILE_M;   // <= max_tiles
    for (int j = tid; j < nt; j += nt_threads) {
        pv.tile_row0[j] = j * TILE_M;
        pv.tile_rows[j] = min(TILE_M, T - j * TILE_M);
        pv.tile_expert[j] = -1;
        pv.tile_rank[j] = 0;
    }
    if (tid == 0) *pv.n_tiles = nt;
    if (pv.decode) {
        for (int t = tid; t < T; t += nt_threads) pv.tok_sorted[t] = t;
        const int nc = min((T + pv.chunk - 1) / pv.chunk, pv.max_groups);
        if (tid == 0) pv.n_groups[0] = pv.n_groups[1] = nc;
        for (int gi = tid; gi < pv.max_groups; gi += nt_threads)
            pv.grp_meta[gi] = gi < nc ? make_int4(-1, gi * pv.chunk, min(T, (gi + 1) * pv.chunk), 0)
                                      : make_int4(-1, 0, 0, 0);
    }
}

// The whole grouping of a batch of at most CAP sequences, by ONE workgroup of PT threads (all of them must
// call it), in LDS.  A device function so that the kernel that routes a request-sized batch can go on to group
// it in the same launch; that kernel hands in LDS it has no more use for.
// Bound by latency: trips to memory, barriers, dependent LDS reads.  The sort is stable and takes the digits
// of the expert alone: up to PLAN_COUNT_S sequences each finds its place by comparing itself with all others
// (one barrier), beyond them a radix sort, 7 bits a pass, lanes of a wave that share a digit finding each other
// with one ballot per bit.  (It was a bitonic sort of 64-bit keys: 36 barriers for 256 sequences, and above
// 2048 through global memory: 8192 sequences took 230 us.)
// IDS_IN_LDS: the caller has left the experts in L.ekey and the offsets in L.off (thread t those of t, t + PT, ..., the last
// offset whichever).
template <int PT, int CAP, bool IDS_IN_LDS = false>
__device__ __forceinline__ void plan_body(const PlanView &pv, const int *seq_offsets, const int *expert_ids,
                                          const int *rank_of_expert, int *err_word, PlanLds<PT, CAP> &L)
{
    using Lds = PlanLds<PT, CAP>;
    static_assert(!IDS_IN_LDS || Lds::KEEPS, "room for the offsets");
    auto offset_of = [&](int s) __attribute__((always_inline)) { return Lds::KEEPS ? L.off[s] : seq_offsets[s]; };
    auto rank_of = [&](int s, int e) __attribute__((always_inline)) {
        return Lds::KEEPS ? L.rank[s] : plan_rank_of(e, rank_of_expert, err_word);
    };
    constexpr bool COMPARES = CAP <= PLAN_CAP_SMALL;   // (the larger instantiation gets no batch that small: less code to fetch, 0.3 us)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int S = pv.S;
    const int T = (int)pv.T;

    // 1. validate, fetch the experts
    if (tid == 0) L.bad_offsets = L.any_long = 0;
    plan_meet<PT>();
    int err = 0;
    if constexpr (!IDS_IN_LDS) {
        if (tid == 0 && (seq_offsets[0] != 0 || seq_offsets[S] != T)) err |= ERR_BAD_OFFSETS;
    } else if (tid == 0 && (L.off[0] != 0 || L.off[S] != T)) {   // (behind the barrier)
        err |= ERR_BAD_OFFSETS;
    }
    for (int s = tid; s < S; s += PT) {
        const int lo = IDS_IN_LDS ? L.off[s] : seq_offsets[s], hi = IDS_IN_LDS ? L.off[s + 1] : seq_offsets[s + 1];
        int e = IDS_IN_LDS ? (int)L.ekey[s] : expert_ids[s];
        if (lo < 0 || hi > T || hi < lo) err |= ERR_BAD_OFFSETS;
        if (e < -1 || e >= pv.E) {
            err |= ERR_BAD_EXPERT;
            e = -1;
        }
        const int rk = plan_rank_of(e, rank_of_expert, err_word);
        if (rk == 0) e = -1;   // rank 0: base model only
        L.ekey[s] = (unsigned)(e + 1);
        L.idx[0][s] = (uint16_t)s;
        if constexpr (Lds::KEEPS) {
            L.rank[s] = rk;
            if constexpr (!IDS_IN_LDS) {
                L.off[s] = lo;
                if (s == S - 1) L.off[S] = hi;
            }
        }
    }
    if (COMPARES && S <= PLAN_COUNT_S && tid < 16 && S + tid < (S + 15) / 16 * 16) L.ekey[S + tid] = ~0u;   // whole turns of the comparison
    if (err) atomicOr(err_word, err);
    if (err & ERR_BAD_OFFSETS) L.bad_offsets = 1;
    plan_plain_tiles(pv, PT);
    plan_meet<PT>();
    if (L.bad_offsets) {
        plan_base_only(pv, PT);
        return;
    }

    // 2. sort the sequences by expert, stably
    int cur = 0;
    if (COMPARES && S <= PLAN_COUNT_S) {
        static_assert(!COMPARES || (PT >= PLAN_COUNT_S && CAP >= PLAN_COUNT_S && PLAN_COUNT_S % 16 == 0), "a sequence per thread");
        if (tid < S) {
            // sixteen keys a turn, four per LDS read: one at a time their latency made it 2.1 us for 64 sequences, now 1.2; of up to
            // eight sequences four a turn (one sequence: 0.15 us less for the kernel)
            const unsigned me = L.ekey[tid];
            int at = 0;
            auto before_me = [&](const uint4 &o, int j) __attribute__((always_inline)) {   // (key k of the four comes first if it is smaller, or equal and k < d)
                const int d = tid - j;
                return (o.x < me + (0 < d)) + (o.y < me + (1 < d)) + (o.z < me + (2 < d)) + (o.w < me + (3 < d));
            };
            auto keys = [&](int j) __attribute__((always_inline)) { return *reinterpret_cast<const uint4 *>(&L.ekey[j]); };
            if (S <= 8) {
                for (int j = 0; j < S; j += 4) at += before_me(keys(j), j);
            } else {
                for (int j = 0; j < S; j += 16) {
                    uint4 o[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[q] = keys(j + 4 * q);
#pragma unroll
                    for (int q = 0; q < 4; ++q) at += before_me(o[q], j + 4 * q);
                }
            }
            L.idx[1][at] = (uint16_t)tid;
        }
        cur = 1;
        plan_meet<PT>();
    } else {
        constexpr int NW = PT / 64;
        const int per_wave = ((S + NW - 1) / NW + 63) / 64 * 64;
        const int w0 = min(wave * per_wave, S), w1 = min(w0 + per_wave, S);
        const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
        for (int shift = 0; shift == 0 || (shift < 32 && ((unsigned)pv.E >> shift) != 0); shift += 7) {
            for (int d = lane; d < 128; d += 64) L.hist[wave][d] = 0;
            for (int i = w0 + lane; i < w1; i += 64)   // (a wave's own row: its LDS operations stay in order)
                atomicAdd(&L.hist[wave][(L.ekey[L.idx[cur][i]] >> shift) & 127], 1);
            plan_meet<PT>();
            // cursors: digits in order, the waves of a digit in order
            constexpr int PER = 128 * NW / PT;   // 2
            int c[PER], v[1] = {0}, total[1];
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int f = tid * PER + q;
                c[q] = L.hist[f % NW][f / NW];
                v[0] += c[q];
            }
            plan_scan<PT, 1>(v, total, L.sums);
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int f = tid * PER + q;
                L.hist[f % NW][f / NW] = v[0];
                v[0] += c[q];
            }
            plan_meet<PT>();
            for (int i = w0 + lane; i - lane < w1; i += 64) {
                const bool ok = i < w1;
                const int s = ok ? L.idx[cur][i] : 0;
                const int d = ok ? (int)((L.ekey[s] >> shift) & 127) : 0;
                uint64_t m = __ballot(ok);
#pragma unroll
                for (int bit = 0; bit < 7; ++bit) {
                    const bool one = (d >> bit) & 1;
                    const uint64_t bal = __ballot(one);
                    m &= one ? bal : ~bal;
                }
                const int base = ok ? L.hist[wave][d] : 0;
                if (ok) {
                    L.idx[cur ^ 1][base + __popcll(m & below)] = (uint16_t)s;
                    if ((m & below) == 0) L.hist[wave][d] = base + __popcll(m);   // the first of them moves the cursor
                }
            }
            cur ^= 1;
            plan_meet<PT>();
        }
    }
    const uint16_t *order = L.idx[cur];
    uint16_t *head_at = L.idx[cur ^ 1];   // per group: its first sorted position

    // 3. tiles / tokens / groups before each sorted position, a run of positions per thread; emit.  (The decode
    // kernels know no tiles, the prefill kernels no token order; a batch that calls may take either way has both.)
    const int per = (S + PT - 1) / PT;
    const int p0 = min(tid * per, S), p1 = min(p0 + per, S);
    int v[3] = {0, 0, 0}, total[3];
    for (int p = p0; p < p1; ++p) {
        const int s = order[p];
        const int len = offset_of(s + 1) - offset_of(s);
        v[0] += (len + TILE_M - 1) / TILE_M;
        v[1] += len;
        v[2] += p == 0 || L.ekey[order[p - 1]] != L.ekey[s];
    }
    plan_scan<PT, 3>(v, total, L.sums);
    if (tid == 0) *pv.n_tiles = pv.tiles ? min(total[0], pv.max_tiles) : 0;
    for (int p = p0; p < p1; ++p) {
        const int s = order[p];
        const int lo = offset_of(s), len = offset_of(s + 1) - lo;
        const int e = (int)L.ekey[s] - 1;
        if (pv.tiles) {
            const int rk = e < 0 ? 0 : rank_of(s, e);   // (a sequence of rank 0 has become one without an adapter)
            for (int left = len, j = 0; left > 0 && v[0] < pv.max_tiles; ++j, ++v[0], left -= TILE_M) {
                pv.tile_row0[v[0]] = lo + j * TILE_M;
                pv.tile_rows[v[0]] = min(left, TILE_M);
                pv.tile_expert[v[0]] = e;
                pv.tile_rank[v[0]] = rk;
            }
        }
        if (pv.decode) {
            L.tokbase[p] = v[1];
            if (p == 0 || L.ekey[order[p - 1]] != L.ekey[s]) head_at[v[2]++] = (uint16_t)p;
            if (len > 8) L.any_long = 1;
            else
                for (int j = 0; j < len && v[1] + j < T; ++j) pv.tok_sorted[v[1] + j] = lo + j;
            v[1] += len;
        }
    }
    if (!pv.decode) return;
    plan_meet<PT>();
    const int n_tok = min(total[1], T), n_groups = total[2];
    if (L.any_long) {
        // The longer sequences: eight lanes each, whole waves for the very long ones.  (A wave for each took 0.11 us a
        // sequence: 500 sequences of up to 24 tokens 26 us for the kernel, now 15.)
        constexpr int NW = PT / 64, WAVE_LEN = 256;
        for (int c = wave * 8; c < S; c += 8 * NW) {
            const int p = c + (lane >> 3);
            const int s = p < S ? order[p] : 0;
            const int lo = p < S ? offset_of(s) : 0, len = p < S ? offset_of(s + 1) - lo : 0;
            const int base = p < S ? L.tokbase[p] : 0;
            if (len > 8 && len <= WAVE_LEN) {
                const int n = min(len, n_tok - base);
                for (int j = lane & 7; j < n; j += 8) pv.tok_sorted[base + j] = lo + j;
            }
            for (uint64_t left = __ballot(len > WAVE_LEN && (lane & 7) == 0); left != 0; left &= left - 1) {
                const int q = __builtin_ctzll(left);
                const int qlo = __builtin_amdgcn_readlane(lo, q), qbase = __builtin_amdgcn_readlane(base, q);
                const int qn = min(__builtin_amdgcn_readlane(len, q), n_tok - qbase);
                for (int j = lane; j < qn; j += 64) pv.tok_sorted[qbase + j] = qlo + j;
            }
        }
    }
    // 4. A group ends where the next one starts.  It is cut into records of at most pv.chunk tokens: the
    // decode kernels hand a record to one column of workgroups, and a hot expert's tokens must not all queue
    // behind one column.
    const int chunk_bits = __builtin_ctz((unsigned)pv.chunk), chunk_m1 = pv.chunk - 1;   // (a power of two: group_chunk)
    const int gper = (n_groups + PT - 1) / PT;
    const int g0 = min(tid * gper, n_groups), g1 = min(g0 + gper, n_groups);
    int n[1] = {0}, n_rec[1];
    for (int g = g0; g < g1; ++g) {
        const int gs = L.tokbase[head_at[g]], ge = g + 1 < n_groups ? L.tokbase[head_at[g + 1]] : n_tok;
        n[0] += (ge - gs + chunk_m1) >> chunk_bits;
    }
    plan_scan<PT, 1>(n, n_rec, L.sums);
    int base_only = 0;
    // Where groups have more than a few records, those of many are written by the whole wave, unless a wave has many such
    // groups: by its own thread the 95 of 6000 base-only tokens took 4 us, but a group for each turn of the wave 64 groups of 8
    // records 8 (600 x 100 tokens: 23.5 us for the kernel, now 15).
    constexpr int FEW_MORE = 8, OWN = 4, SHARED_GROUPS = 8, OWN_MOST = 64;
    if (n_rec[0] - n_groups <= FEW_MORE) {
        for (int g = g0; g < g1; ++g) {
            const int p = head_at[g], s = order[p];
            const int gs = L.tokbase[p], ge = g + 1 < n_groups ? L.tokbase[head_at[g + 1]] : n_tok;
            const int e = (int)L.ekey[s] - 1;
            const int rk = e >= 0 ? rank_of(s, e) : 0;   // (a sequence of rank 0 has become one without an adapter)
            for (int t = gs; t < ge && n[0] < pv.max_groups; t += pv.chunk, ++n[0])
                pv.grp_meta[n[0]] = make_int4(e, t, min(t + pv.chunk, ge), rk);
            if (e < 0) base_only = n[0];   // (the first group, if any)
        }
    } else {
        for (int k = 0; k < gper; ++k) {   // (the same number of turns for the whole wave)
            const int g = g0 + k;
            int e = -1, rk = 0, gs = 0, ge = 0;
            if (g < g1) {
                const int p = head_at[g], s = order[p];
                gs = L.tokbase[p];
                ge = g + 1 < n_groups ? L.tokbase[head_at[g + 1]] : n_tok;
                e = (int)L.ekey[s] - 1;
                if (e >= 0) rk = rank_of(s, e);
            }
            const int recs = (ge - gs + chunk_m1) >> chunk_bits, first = n[0];
            const int own = __popcll(__ballot(recs > OWN)) <= SHARED_GROUPS ? OWN : OWN_MOST;
            if (recs <= own)
                for (int j = 0; j < recs && first + j < pv.max_groups; ++j)
                    pv.grp_meta[first + j] = make_int4(e, gs + (j << chunk_bits), min(gs + ((j + 1) << chunk_bits), ge), rk);
            for (uint64_t left = __ballot(recs > own); left != 0; left &= left - 1) {
                const int q = __builtin_ctzll(left);
                const int qe = __builtin_amdgcn_readlane(e, q), qrk = __builtin_amdgcn_readlane(rk, q);
                const int qs = __builtin_amdgcn_readlane(gs, q), qend = __builtin_amdgcn_readlane(ge, q);
                const int qfirst = __builtin_amdgcn_readlane(first, q), qn = __builtin_amdgcn_readlane(recs, q);
                for (int j = lane; j < qn && qfirst + j < pv.max_groups; j += 64)
                    pv.grp_meta[qfirst + j] = make_int4(qe, qs + (j << chunk_bits), min(qs + ((j + 1) << chunk_bits), qend), qrk);
            }
            n[0] = min(first + recs, max(first, pv.max_groups));
            if (g < g1 && e < 0) base_only = n[0];
        }
    }
    const int n_out = min(n_rec[0], pv.max_groups);
    if (tid == 0) {
        pv.n_groups[0] = n_out;
        pv.n_groups[1] = base_only;
    }
    // unused records read as empty groups, so the decode kernels need not
    // fetch the group count before their own record
    for (int gi = n_out + tid; gi < pv.max_groups; gi += PT) pv.grp_meta[gi] = make_int4(-1, 0, 0, 0);
}

}  // namespace moin
