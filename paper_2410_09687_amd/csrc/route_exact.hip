// Nearest-topic search by the squared distance itself (Section 3.3), written out as the sum of squared
// differences in fp32: fp32 embeddings in moin_route, both storage types in moin_route_topk ("Future
// Works", creating new experts on the fly: the k nearest topics of a query).
//
// Every distance is computed in ONE way, whichever kernel does it and wherever the pair lies: lane l of a
// wave sums the 16-byte chunks l, l + 64, ... of the two rows, and the 64 partial sums meet in a fixed tree
// (lanes 32 apart, then 16, 8, 4, 2, 1).  Equal centroids therefore get equal bits, and "lowest index wins a
// tie" holds across kernels.
//
//  * route_direct_kernel: every pair of a small problem.  A wave takes 8 queries x 8 centroids at a time (64
//    sums in registers, 16 loads of 16 bytes per lane for 512 vector instructions), waves split the
//    centroids, the winners meet in the packed 64-bit atomic minimum of the small-batch bf16 router.
//  * route_screen_kernel + route_pick_kernel: for larger problems the distances are first bounded by a bf16
//    MFMA product -- fp32 values as a sum of two bf16, three products -- of which only the smallest score of
//    every group of 16 centroids leaves the workgroup; a wave per query then computes the exact distances of
//    the groups that can hold one of its k nearest centroids, by a bound on what the screening arithmetic
//    can be wrong by.  The answer is that of the exhaustive search, bit for bit.
#include <algorithm>
#include <type_traits>

#include "gemm_core.h"
#include "kernels.h"
#include "route_finish.h"
#include "wave_sums.h"

namespace moin {

namespace {

template <bool BF16>
struct Vals {
    static constexpr int N = BF16 ? 8 : 4;   // values per 16-byte chunk
    __device__ static __forceinline__ void unpack(const uint4 &v, float (&f)[N])
    {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if constexpr (BF16) {
                f[2 * t] = bits_f32(w[t] << 16);
                f[2 * t + 1] = bits_f32(w[t] & 0xFFFF0000u);
            } else {
                f[t] = bits_f32(w[t]);
            }
        }
    }
};

// 64 sums over the wave at once; lane l returns the sum of a[l].
__device__ __forceinline__ float wave_sums(float (&a)[64], int lane)
{
#pragma unroll
    for (int j = 0; j < 32; ++j) a[j] = merge32(a[j], a[j + 32]);
#pragma unroll
    for (int j = 0; j < 16; ++j) a[j] = merge16(a[j], a[j + 16]);
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = merge_x<8>(a[j], a[j + 8], lane);
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = merge_x<4>(a[j], a[j + 4], lane);
#pragma unroll
    for (int j = 0; j < 2; ++j) a[j] = merge_x<2>(a[j], a[j + 2], lane);
    return merge_x<1>(a[0], a[1], lane);
}

typedef unsigned long long u64;
constexpr u64 NO_KEY = ~0ull;

// (distance, index) as an integer that orders like the pair: distances are sums of squares, never below zero.
__device__ __forceinline__ u64 dist_key(float d, int c) { return ((u64)f32_bits(d) << 32) | (unsigned)c; }

__device__ __forceinline__ u64 shfl_xor64(u64 v, int m)
{
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, m), hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), m);
    return ((u64)hi << 32) | lo;
}
__device__ __forceinline__ u64 readlane64(u64 v, int l)
{
    return ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
}

}  // namespace

// ---- every pair of a small fp32 problem ---------------------------------------------------------------------

// Bound by latency on the sizes it is chosen for (a launch, two trips to memory, the exchange of winners);
// 8 x 8 pairs per wave keep the vector unit, not the loads, ahead of what remains.  7 x 500 x 384: 760 us with
// one wave per query walking the centroids one by one, 13 us here.
// Wave w of the grid: queries 8 (w / n_runs) .. + 8 against centroid batches (of 8) [run * per, ...).
__global__ __launch_bounds__(256) void route_direct_kernel(RouteKParams p, int n_runs, int per, int retained_only)
{
    using V = Vals<false>;
    extern __shared__ __align__(16) char smem[];   // for the grouping alone
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t)blockIdx.x * 4 + uniform(threadIdx.x >> 6);
    const int64_t q0 = w / n_runs * 8;
    const int run = (int)(w % n_runs);
    const int ncb = (p.K + 7) / 8;
    if (q0 < p.N) {
        const int64_t row_bytes = (int64_t)p.D * 4;
        const int nch = p.D / V::N;
        const char *q[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) q[i] = p.emb + (q0 + i < p.N ? q0 + i : p.N - 1) * row_bytes;
        float bv = __builtin_inff();
        int bi = 0;
        for (int b = run * per; b < min(ncb, run * per + per); ++b) {
            const char *c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = p.cent + (int64_t)min(b * 8 + u, p.K - 1) * row_bytes;
            float acc[64];
#pragma unroll
            for (int j = 0; j < 64; ++j) acc[j] = 0.f;
            for (int ch = lane; ch < nch; ch += 64) {
                uint4 vq[8], vc[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) vc[u] = *reinterpret_cast<const uint4 *>(c[u] + (int64_t)ch * 16);
#pragma unroll
                for (int i = 0; i < 8; ++i) vq[i] = *reinterpret_cast<const uint4 *>(q[i] + (int64_t)ch * 16);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    float x[V::N];
                    V::unpack(vq[i], x);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        float y[V::N];
                        V::unpack(vc[u], y);
#pragma unroll
                        for (int t = 0; t < V::N; ++t) {
                            const float df = x[t] - y[t];
                            acc[i * 8 + u] = fmaf(df, df, acc[i * 8 + u]);
                        }
                    }
                }
            }
            const float d = wave_sums(acc, lane);   // lane: query lane / 8, centroid lane % 8 of the batch
            const int ci = b * 8 + (lane & 7);
            if (ci < p.K && !(retained_only && p.slot[ci] < 0) && d < bv) {   // (a NaN never wins)
                bv = d;
                bi = ci;
            }
        }
        u64 key = bv < __builtin_inff() ? dist_key(bv, bi) : NO_KEY;
#pragma unroll
        for (int m = 4; m > 0; m >>= 1) {
            const u64 o = shfl_xor64(key, m);
            key = o < key ? o : key;
        }
        const int64_t qi = q0 + (lane >> 3);
        if ((lane & 7) == 0 && qi < p.N && key != NO_KEY) atomicMin(&p.best[qi], key);
    }
    if (p.finish) route_finish<256>(p, smem);
}

// ---- screening ---------------------------------------------------------------------------------------------

struct ScreenKParams {
    const char *cent, *emb;    // rows as they came
    char *cent_p, *emb_p;      // bf16 planes of Dp values (fp32: of every 32 values the high parts, then the remainders;
                               // bf16 with D % 64: the values padded with zeros), or the rows themselves
    float *cnorm, *qnorm;      // ||.||^2; cnorm [nct * 128], +inf for what takes no part in the search
    float *cmax;               // [nct] largest finite cnorm of a tile
    float *minima;             // [n, 8 nct] smallest ||c||^2 - 2 q.c of every group of 16 centroids
    int *counts;               // [K] or null: zeroed by the preparation
    const int *slot;
    int retained_only;
    int64_t n;                 // queries of this part of the batch
    int K, D, Dp, nct;
    int planes;                // 2: fp32, 1: bf16 padded, 0: bf16 used as it is
    int with_cent;             // the preparation does the centroids too (first part of a batch)
};

// One wave per row: its squared norm, and its bf16 planes where the rows cannot be used as they are.
template <bool BF16>
__global__ __launch_bounds__(256) void route_prep_kernel(ScreenKParams p)
{
    const int lane = threadIdx.x & 63;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p.counts && gid < p.K) p.counts[gid] = 0;   // (the grid has at least K threads: a wave per centroid)
    const int n_cent = p.with_cent ? p.nct * 128 : 0;
    int64_t row = (int64_t)blockIdx.x * 4 + uniform(threadIdx.x >> 6);
    const bool is_cent = row < n_cent;
    if (!is_cent) row -= n_cent;
    if (!is_cent && row >= p.n) return;
    float *norm = is_cent ? p.cnorm : p.qnorm;
    if (is_cent && row >= p.K) {
        if (lane == 0) norm[row] = __builtin_inff();
        return;
    }
    const char *src = (is_cent ? p.cent : p.emb) + row * (int64_t)p.D * (BF16 ? 2 : 4);
    const int64_t pitch = (int64_t)p.Dp * 2 * p.planes;
    char *dst = (is_cent ? p.cent_p : p.emb_p) + row * pitch;
    float sum = 0.f;
    for (int ch = lane; ch < p.Dp / 8; ch += 64) {   // 8 values
        float f[8];
        uint4 raw = make_uint4(0, 0, 0, 0);
        if constexpr (BF16) {
            if (ch * 8 < p.D) raw = *reinterpret_cast<const uint4 *>(src + ch * 16);   // D % 8 == 0
            Vals<true>::unpack(raw, f);
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {                                              // D % 4 == 0
                uint4 v = make_uint4(0, 0, 0, 0);
                if (ch * 8 + h * 4 < p.D) v = *reinterpret_cast<const uint4 *>(src + ch * 32 + h * 16);
                f[4 * h] = bits_f32(v.x); f[4 * h + 1] = bits_f32(v.y);
                f[4 * h + 2] = bits_f32(v.z); f[4 * h + 3] = bits_f32(v.w);
            }
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) sum = fmaf(f[t], f[t], sum);
        if (p.planes == 0) continue;
        if constexpr (BF16) {
            *reinterpret_cast<uint4 *>(dst + ch * 16) = raw;
        } else {
            uint32_t h[4], l[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                h[t] = pack_bf16x2(f[2 * t], f[2 * t + 1]);
                l[t] = pack_bf16x2(f[2 * t] - bits_f32(h[t] << 16), f[2 * t + 1] - bits_f32(h[t] & 0xFFFF0000u));
            }
            char *at = dst + (ch >> 2) * 128 + (ch & 3) * 16;
            *reinterpret_cast<uint4 *>(at) = make_uint4(h[0], h[1], h[2], h[3]);
            *reinterpret_cast<uint4 *>(at + 64) = make_uint4(l[0], l[1], l[2], l[3]);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if (is_cent) {
        if (p.retained_only && p.slot[row] < 0) sum = __builtin_inff();
        else if (!(sum < __builtin_inff())) sum = 3.4e38f;   // overflow or NaN: takes part, the bound below gives up on it
    }
    if (lane == 0) norm[row] = sum;
}

// Matrix product bound by its short contraction (6 to 12 blocks of 64 per tile) and, in the fp32 case, by three
// times its flops; what leaves is 1/16 of the scores.  1000 x 5000 x 384, fp32: 8100 us for the exhaustive
// search with one wave per query; 6 + 18 + 11 us for preparation, screening and exact distances.  The same with
// 768 dimensions in bf16 and the four nearest: 1400 us against 4 + 15 + 22 us.
// 128 centroids x 128 queries per workgroup, four waves of 64 x 64, two workgroups per compute unit.
using CfgScreen = DmaCore<128, 128, 64, 2, 2, 2>;

// fp32: a block is the high parts of 32 values, then their remainders, and gives all three products (high x high, high x
// remainder, remainder x high) from one load into LDS: two thirds of the blocks, barriers, bytes and LDS reads of three
// passes.  Us of a call, three passes / this: 1000 x 5000 x 384 33.0 / 32.4, 16 000 queries 255 / 231, by 768 500 / 442,
// 100 x 5000 x 768 43.7 / 36.8, 70 000 x 1000 x 96 207 / 199.
struct CfgScreenPairs : CfgScreen {
    __device__ static __forceinline__ void compute_stage(const char *stage, Acc &acc)
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int wm = wave / WN, wn = wave % WN;
        const int r = lane & 31, h = lane >> 5, f = swz(r);
        __builtin_amdgcn_iglp_opt(1);   // (16 000 x 5000 x 384: without it 234 us instead of 228)
        const char *pa = stage + (wm * WTM + r) * ROWB;
        const char *pb = stage + A_BYTES + (wn * WTN + r) * ROWB;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8_t a[2][FM], b[2][FN];   // high parts, remainders
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int o = ((q * 4 + ks * 2 + h) ^ f) * 16;
#pragma unroll
                for (int i = 0; i < FM; ++i)
                    a[q][i] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(pa + i * 32 * ROWB + o));
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    b[q][j] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(pb + j * 32 * ROWB + o));
            }
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        acc.v[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[q == 2][i], b[q == 1][j], acc.v[i][j], 0, 0, 0);
        }
    }
};

// by_cent: the tiles of one centroid tile are neighbours, so that an XCD reads an eighth of the centroids and every query,
// where those are the fewer.  Us of a call, by query tile / by centroid tile: fp32 1000 x 5000 x 384 35 / 32.5, 2500 51.8 / 51.2, 4500
// 76.6 both, 5500 88.4 both, 10 000 148.5 / 149.5, 16 000 254 / 276, 750 x 1500 24.3 / 24.0, 2250 27.1 / 27.6; bf16 with the
// four nearest 2500 x 5000 x 768 65.4 / 63.6, 4500 95.0 / 94.7, 5500 109.8 / 111.7, 10 000 180 / 195.
template <bool PAIRS>
__global__ __launch_bounds__(CfgScreen::NT) void route_screen_kernel(ScreenKParams p, int nqt, int by_cent)
{
    using C = std::conditional_t<PAIRS, CfgScreenPairs, CfgScreen>;
    extern __shared__ __align__(16) char smem[];
    const int id = xcd_band_id(blockIdx.x, nqt * p.nct);
    if (id < 0) return;
    const int qt = uniform(by_cent ? id % nqt : id / p.nct), ct = uniform(by_cent ? id / nqt : id % p.nct);
    const int64_t q0 = (int64_t)qt * C::BN;
    const int nq = (int)min((int64_t)C::BN, p.n - q0), nc = min(C::BM, p.K - ct * C::BM);
    const uint32_t ld = (uint32_t)p.Dp * (PAIRS ? 4u : 2u);
    const char *cb = p.cent_p + (int64_t)ct * C::BM * ld, *qb = p.emb_p + q0 * (int64_t)ld;
    const auto lc = C::template make_lanes<C::A_I>(nc);
    const auto lq = C::template make_lanes<C::B_I>(nq);
    typename C::Acc acc;
    C::zero(acc);
    auto issue = [=](int b, char *stage) __attribute__((always_inline)) {
        C::issue(stage, cb, ld, lc, qb, ld, lq, (uint32_t)b * C::ROWB);
    };
    dma_pipelined_blocks<C>(smem, (int)(ld / C::ROWB), issue, acc, [](int) {});

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / C::WN, wn = wave % C::WN;
    if (qt == 0 && wave == 0) {
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float v = p.cnorm[ct * 128 + i * 64 + lane];
            if (v < __builtin_inff()) m = fmaxf(m, v);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
        if (lane == 0) p.cmax[ct] = m;
    }
    // a lane holds 16 centroids of one query per accumulator: one group
    float g[C::FM][C::FN];
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < C::FN; ++j) g[i][j] = __builtin_inff();
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            const f32x4_t c4 = *reinterpret_cast<const f32x4_t *>(p.cnorm + ct * 128 + wm * C::WTM + i * 32 + e4 * 8 +
                                                                  4 * (lane >> 5));
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < C::FN; ++j) g[i][j] = fminf(g[i][j], fmaf(-2.f, acc.v[i][j][e4 * 4 + q], c4[q]));
        }
    static_assert(C::FM == 2, "four groups per lane pair below");
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
        const float o0 = __shfl_xor(g[0][j], 32), o1 = __shfl_xor(g[1][j], 32);
        const int col = wn * C::WTN + j * 32 + lane;
        if (lane < 32 && col < nq)
            *reinterpret_cast<f32x4_t *>(p.minima + (q0 + col) * (8 * (int64_t)p.nct) + ct * 8 + wm * 4) =
                f32x4_t{g[0][j], o0, g[1][j], o1};
    }
}

// ---- exact distances of a query's candidates ---------------------------------------------------------------

struct PickKParams {
    const char *emb, *cent;
    const float *minima;       // null: every centroid is a candidate
    const float *qnorm, *cmax;
    const int *slot;
    int retained_only;
    int64_t n;
    int K, D, nct, k;
    float err_dot;             // |error of the screened q.c| <= err_dot ||q|| ||c||
    float err_rel;             // relative error of an fp32 sum of D squares
    int *cid, *expert_ids;     // [n, k] or null
    float *d2;                 // [n, k] or null
    int *counts;               // [K] or null
    int none_id;               // the id of a place that nothing fills
};

// W waves per query (W = 1: four queries per workgroup).  Group g: the centroids 32 (g / 2) + 8 a + 4 (g % 2) + b,
// a, b = 0..3 -- the rows a lane of the screening kernel holds.  The list of the k best so far: lane m holds place m.
template <bool BF16, int W>
__global__ __launch_bounds__(W == 1 ? 256 : 64 * W) void route_pick_kernel(PickKParams p)
{
    using V = Vals<BF16>;
    __shared__ u64 lists[W][8];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int64_t qi = W == 1 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x;
    if (qi >= p.n) return;
    const int64_t row_bytes = (int64_t)p.D * (BF16 ? 2 : 4);
    const char *q = p.emb + qi * row_bytes;
    const int nch = p.D / V::N;
    const int n_groups = 2 * ((p.K + 31) / 32);
    const float *mins = p.minima ? p.minima + qi * (8 * (int64_t)p.nct) : nullptr;

    // A group can hold one of the k nearest only if its smallest screened score is at most `thr`.  With eps the
    // largest error of a screened score and delta the relative error of a computed distance: some k centroids
    // have a screened score of at most M, hence a computed distance of at most (M + eps + ||q||^2) (1 + delta);
    // whatever is among the k nearest has one no larger, hence a screened score of at most
    // (M + eps + ||q||^2) (1 + delta) / (1 - delta) - ||q||^2 + eps.
    // (eps is that of the longest centroid: one of a thousand times the others' length, or one that is no number, and
    // every group stays a candidate.  1000 x 5000 x 384 in fp32 then takes 643 us instead of 37.)
    float thr = __builtin_inff();
    if (mins) {
        float m = __builtin_inff();
        for (int g = lane; g < n_groups; g += 64) m = fminf(m, mins[g]);
        float M = __builtin_inff();
        u64 key = ((u64)(f32_bits(m) & 0x80000000u ? ~f32_bits(m) : f32_bits(m) | 0x80000000u) << 32) | (unsigned)lane;
        for (int r = 0; r < p.k; ++r) {   // the k-th smallest of the lanes' minima: k different groups lie at or below it
            u64 best = key;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const u64 v = shfl_xor64(best, o);
                best = v < best ? v : best;
            }
            M = __shfl(m, (int)(best & 63));
            if (key == best) key = NO_KEY;
        }
        float c2 = 0.f;
        for (int t = lane; t < p.nct; t += 64) c2 = fmaxf(c2, p.cmax[t]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) c2 = fmaxf(c2, __shfl_xor(c2, o));
        const float q2 = p.qnorm[qi];
        if (q2 < 1e37f && c2 < 1e37f) {   // beyond (or NaN) the bound says nothing: every group is looked at
            const float eps = 2.f * p.err_dot * sqrtf(q2) * sqrtf(c2) + p.err_rel * (c2 + q2) + 1e-30f;
            thr = M + 2.f * eps + 4.f * p.err_rel * fmaxf(M + eps + q2, 0.f);
        }
    }

    u64 list = NO_KEY;
    int turn = 0;
    for (int gb = 0; gb < n_groups; gb += 64) {
        const bool cand = gb + lane < n_groups && !(mins && mins[gb + lane] > thr);
        for (u64 mask = __ballot(cand); mask; mask &= mask - 1) {
            if (W > 1 && (turn++ % W) != wave) continue;
            const int g = gb + __ffsll((unsigned long long)mask) - 1;
            const int c_first = 32 * (g >> 1) + 4 * (g & 1);
            const char *c[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) c[t] = p.cent + (int64_t)min(c_first + 8 * (t >> 2) + (t & 3), p.K - 1) * row_bytes;
            float acc[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) acc[t] = 0.f;
            for (int ch = lane; ch < nch; ch += 64) {
                uint4 vc[16];
                const uint4 vq = *reinterpret_cast<const uint4 *>(q + (int64_t)ch * 16);
#pragma unroll
                for (int t = 0; t < 16; ++t) vc[t] = *reinterpret_cast<const uint4 *>(c[t] + (int64_t)ch * 16);
                float x[V::N];
                V::unpack(vq, x);
#pragma unroll
                for (int t = 0; t < 16; ++t) {
                    float y[V::N];
                    V::unpack(vc[t], y);
#pragma unroll
                    for (int j = 0; j < V::N; ++j) {
                        const float df = x[j] - y[j];
                        acc[t] = fmaf(df, df, acc[t]);
                    }
                }
            }
            const float d = wave_sums(acc, lane);
            const int ci = c_first + 8 * (lane >> 4) + ((lane >> 2) & 3);
            const bool ok = ci < p.K && !(p.retained_only && p.slot[ci] < 0) && d < __builtin_inff();
            const u64 key = ok ? dist_key(d, ci) : NO_KEY;
            // enter, one by one, what beats the list's last place
            u64 last = readlane64(list, p.k - 1);
            for (u64 m2 = __ballot(key < last && (lane & 3) == 0); m2; m2 &= m2 - 1) {
                const u64 x = readlane64(key, __ffsll((unsigned long long)m2) - 1);
                if (!(x < last)) continue;
                const int at = __popcll(__ballot(list < x && lane < p.k));
                const u64 up = ((u64)(uint32_t)__shfl_up((int)(uint32_t)(list >> 32), 1) << 32) |
                               (uint32_t)__shfl_up((int)(uint32_t)list, 1);
                list = lane < at ? list : (lane == at ? x : up);
                last = readlane64(list, p.k - 1);
            }
        }
    }
    if constexpr (W > 1) {
        if (lane < p.k) lists[wave][lane] = list;
        __syncthreads();
        if (wave != 0) return;
        u64 last = readlane64(list, p.k - 1);
        for (int w = 1; w < W; ++w)
            for (int m = 0; m < p.k; ++m) {
                const u64 x = lists[w][m];   // the same for the whole wave
                if (!(x < last)) break;      // (each list is in order)
                const int at = __popcll(__ballot(list < x && lane < p.k));
                const u64 up = ((u64)(uint32_t)__shfl_up((int)(uint32_t)(list >> 32), 1) << 32) |
                               (uint32_t)__shfl_up((int)(uint32_t)list, 1);
                list = lane < at ? list : (lane == at ? x : up);
                last = readlane64(list, p.k - 1);
            }
    }
    if (lane < p.k) {
        const bool filled = list != NO_KEY;
        const int c = filled ? (int)(list & 0xffffffffu) : p.none_id;
        const int64_t at = qi * p.k + lane;
        if (p.cid) p.cid[at] = c;
        if (p.expert_ids) p.expert_ids[at] = c < 0 ? -1 : (p.slot ? p.slot[c] : c);
        if (p.d2) p.d2[at] = filled ? bits_f32((uint32_t)(list >> 32)) : __builtin_inff();
        if (p.counts) atomicAdd(&p.counts[c], 1);
    }
}

// ---- launches ----------------------------------------------------------------------------------------------

// Pairs x dimension from which screening (three launches) beats computing every distance.  Measured in us a
// call, direct / screened: 300 x 500 x 384 (58 M) 14 / 29, 306 x 1421 x 256 (111 M) 20 / 30, 1000 x 500 x 384
// (192 M) 27 / 27; 1000 x 5000 x 384 (1.9 G) 150 / 35.
constexpr int64_t SCREEN_MIN_WORK = 150'000'000;
// With fewer centroids the screen's tiles of 128 are half padding and three launches have little to save (moin_route, us
// direct / screened: 262144 queries x 16 x 384 163 / 759, x 64 549 / 788, 2000 x 200 x 768 35 / 46); large batches would
// gain from about 128 on (262144 x 128 x 384 1018 / 802, x 200 1495 / 831), small ones lose up to here (2000 x 255 x 768
// 38 / 46).
constexpr int SCREEN_MIN_K = 256;
// moin_route_topk: with this many centroids even one query gains, since its eight waves then take more than eight
// turns of 16 centroids, 3.6 us each (1 query, every distance / screened: 1030 x 384 28 / 23 in bf16, 29 / 31 in
// fp32; 1500 x 768 48 / 30 and 56 / 48; 5000 x 768 144 / 34 and 163 / 55; 100000 x 384 1747 / 92 and 2055 / 144).
constexpr int TOPK_SCREEN_MIN_K = 1024;
// Queries screened at a time: at most this many, 64 MiB of group minima (which grow with K) and 128 MiB of planes
// (which grow with D), but 128 at least.  The centroids' planes are a copy of the whole table.
constexpr int64_t SCREEN_QUERIES = 32768, SCREEN_MINIMA_BYTES = 64 << 20, SCREEN_PLANES_BYTES = 128 << 20;

bool route_direct_small(int64_t N, int K, int D, int is_bf16)
{
    return !is_bf16 && N <= ROUTE_SMALL_MAX_N && N * K <= SCREEN_MIN_WORK / D;
}

bool route_screen_pays(int64_t N, int K, int D, bool topk)
{
    if (N <= 0) return false;
    if (topk && K > TOPK_SCREEN_MIN_K) return true;
    return K >= SCREEN_MIN_K && (double)N * K * D > (double)SCREEN_MIN_WORK;
}

struct ScreenLayout {
    int Dp, nct, planes;
    int64_t part;
    size_t cent_p, emb_p, cnorm, qnorm, cmax, minima, total;
};

static ScreenLayout screen_layout(int64_t N, int K, int D, int is_bf16)
{
    ScreenLayout L;
    L.Dp = (D + 63) / 64 * 64;
    L.nct = (K + 127) / 128;
    L.planes = is_bf16 ? (L.Dp == D ? 0 : 1) : 2;
    int64_t part = std::min(SCREEN_QUERIES, SCREEN_MINIMA_BYTES / ((int64_t)L.nct * 32));
    if (L.planes) part = std::min(part, SCREEN_PLANES_BYTES / ((int64_t)L.Dp * 2 * L.planes));
    part = std::max<int64_t>(128, part / 128 * 128);
    L.part = N < part ? N : part;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += (bytes + 255) / 256 * 256;
        return at;
    };
    L.cnorm = take((size_t)L.nct * 128 * 4);
    L.qnorm = take((size_t)L.part * 4);
    L.cmax = take((size_t)L.nct * 4);
    L.minima = take((size_t)L.part * L.nct * 32);
    L.cent_p = take((size_t)K * L.Dp * 2 * L.planes);
    L.emb_p = take((size_t)L.part * L.Dp * 2 * L.planes);
    L.total = off;
    return L;
}

size_t route_screen_bytes(int64_t N, int K, int D, int is_bf16) { return screen_layout(N, K, D, is_bf16).total; }

// Waves per query behind a screen.  The k nearest lie in about k groups, a trip to memory each: several waves take them side
// by side as long as the chip has room for them.  Us a call, one / two / four waves: 100 x 5000 x 768 bf16, k = 4, 38 / 31 / 29,
// 1000 queries 45 / 40 / 39, 2000 61 / 58 / 65, 3000 71 / 75 / 82; 2000 x 3000 x 384 fp32, k = 8, 62 / 58 / 64.  A single
// nearest centroid lies in one group or two: 1000 x 5000 x 384 fp32 35 / 34.5 / 35, 2500 57 / 57 / 63.
static int pick_waves(int64_t n, int k)
{
    if (k == 1) return 1;
    return n <= 4 * compute_units() ? 4 : n <= 8 * compute_units() ? 2 : 1;
}

template <bool BF16>
static void launch_pick(const PickKParams &p, int waves, hipStream_t stream)
{
    if (waves >= 8) hipLaunchKernelGGL((route_pick_kernel<BF16, 8>), dim3((unsigned)p.n), dim3(512), 0, stream, p);
    else if (waves == 4) hipLaunchKernelGGL((route_pick_kernel<BF16, 4>), dim3((unsigned)p.n), dim3(256), 0, stream, p);
    else if (waves == 2) hipLaunchKernelGGL((route_pick_kernel<BF16, 2>), dim3((unsigned)p.n), dim3(128), 0, stream, p);
    else hipLaunchKernelGGL((route_pick_kernel<BF16, 1>), dim3((unsigned)((p.n + 3) / 4)), dim3(256), 0, stream, p);
}

static PickKParams pick_params(const RouteArgs &a, int k, float *d2, int none_id)
{
    PickKParams p;
    p.emb = (const char *)a.emb; p.cent = (const char *)a.cent;
    p.minima = nullptr; p.qnorm = nullptr; p.cmax = nullptr;
    p.slot = a.slot; p.retained_only = a.retained_only;
    p.n = a.N; p.K = a.K; p.D = a.D; p.nct = (a.K + 127) / 128; p.k = k;
    p.err_dot = p.err_rel = 0.f;
    p.cid = a.cid; p.expert_ids = a.expert_ids; p.d2 = d2; p.counts = nullptr;
    p.none_id = none_id;
    return p;
}

hipError_t launch_route_screened(const RouteArgs &a, int k, float *d2, int none_id, void *ws, hipStream_t stream)
{
    const ScreenLayout L = screen_layout(a.N, a.K, a.D, a.is_bf16);
    char *w = static_cast<char *>(ws);
    ScreenKParams s;
    s.cent = (const char *)a.cent;
    s.cent_p = L.planes ? w + L.cent_p : (char *)a.cent;
    s.cnorm = reinterpret_cast<float *>(w + L.cnorm);
    s.qnorm = reinterpret_cast<float *>(w + L.qnorm);
    s.cmax = reinterpret_cast<float *>(w + L.cmax);
    s.minima = reinterpret_cast<float *>(w + L.minima);
    s.slot = a.slot; s.retained_only = a.retained_only;
    s.K = a.K; s.D = a.D; s.Dp = L.Dp; s.nct = L.nct; s.planes = L.planes;
    PickKParams p = pick_params(a, k, d2, none_id);
    p.minima = s.minima; p.qnorm = s.qnorm; p.cmax = s.cmax;
    p.counts = a.counts;
    // Screened product: fp32 values as h + l with |x - h| <= 2^-9 |x|, |x - h - l| <= 2^-18 |x|, the product
    // l l left out: at most 3.1 * 2^-18 of ||q|| ||c|| (Cauchy-Schwarz); fp32 accumulation of n products,
    // at most n half-ulps each taken as a whole one.  bf16 values: the products are exact.
    const double u = 1.0 / (1 << 23);
    p.err_dot = (float)((a.is_bf16 ? 0.0 : 3.2 / (1 << 18)) + 1.02 * ((L.planes == 2 ? 3 : 1) * (double)L.Dp + 64) * u);
    p.err_rel = (float)((a.D / 64 + 24) * u);
    const int64_t row_bytes = (int64_t)a.D * (a.is_bf16 ? 2 : 4);
    for (int64_t q = 0; q < a.N; q += L.part) {
        s.n = p.n = a.N - q < L.part ? a.N - q : L.part;
        s.emb = p.emb = (const char *)a.emb + q * row_bytes;
        s.emb_p = L.planes ? w + L.emb_p : (char *)s.emb;
        s.with_cent = q == 0;
        s.counts = q == 0 ? a.counts : nullptr;
        const int64_t rows = (s.with_cent ? (int64_t)L.nct * 128 : 0) + s.n;
        const dim3 pg((unsigned)((rows + 3) / 4));
        if (a.is_bf16) hipLaunchKernelGGL(route_prep_kernel<true>, pg, dim3(256), 0, stream, s);
        else hipLaunchKernelGGL(route_prep_kernel<false>, pg, dim3(256), 0, stream, s);
        const int nqt = (int)((s.n + 127) / 128);
        const int64_t grid = ((int64_t)nqt * L.nct + 7) / 8 * 8;
        if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
        const int by_cent = s.n < s.K ? 1 : 0;
        if (L.planes == 2)
            hipLaunchKernelGGL(route_screen_kernel<true>, dim3((unsigned)grid), dim3(CfgScreen::NT), CfgScreen::SMEM_BYTES, stream,
                               s, nqt, by_cent);
        else
            hipLaunchKernelGGL(route_screen_kernel<false>, dim3((unsigned)grid), dim3(CfgScreen::NT), CfgScreen::SMEM_BYTES, stream,
                               s, nqt, by_cent);
        if (a.is_bf16) launch_pick<true>(p, pick_waves(p.n, p.k), stream);
        else launch_pick<false>(p, pick_waves(p.n, p.k), stream);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (p.cid) p.cid += s.n * k;
        if (p.expert_ids) p.expert_ids += s.n * k;
        if (p.d2) p.d2 += s.n * k;
    }
    return hipSuccess;
}

// All pairs of fp32 embeddings; p.finish: the last workgroup turns the packed minima into ids.
hipError_t launch_route_direct(const RouteKParams &p, int retained_only, hipStream_t stream)
{
    const int64_t nqb = (p.N + 7) / 8;
    const int64_t ncb = (p.K + 7) / 8;
    // about 4096 waves, each at least one batch of eight centroids
    int64_t runs = nqb >= 4096 ? 1 : 4096 / nqb;
    if (runs > ncb) runs = ncb;
    const int64_t per = (ncb + runs - 1) / runs;
    runs = (ncb + per - 1) / per;
    const int64_t grid = (nqb * runs + 3) / 4;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(route_direct_kernel, dim3((unsigned)grid), dim3(256),
                       p.with_plan ? sizeof(PlanLdsSmall) : 0, stream, p, (int)runs, (int)per,
                       retained_only);
    return hipGetLastError();
}

// The k nearest centroids of every query (ws: null, or route_screen_bytes() of device memory).
hipError_t launch_route_topk(const RouteArgs &a, int k, float *d2, void *ws, hipStream_t stream)
{
    if (a.N <= 0) return hipSuccess;
    if (k < 1 || k > 8 || a.N > 0x7fffffffLL) return hipErrorInvalidValue;
    if (ws) return launch_route_screened(a, k, d2, -1, ws, stream);
    const PickKParams p = pick_params(a, k, d2, -1);
    const int waves = a.N < 2048 ? 8 : 1;   // few queries: several waves share one
    if (a.is_bf16) launch_pick<true>(p, waves, stream);
    else launch_pick<false>(p, waves, stream);
    return hipGetLastError();
}

hipError_t prepare_route_exact_kernels()
{
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&route_screen_kernel<false>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, CfgScreen::SMEM_BYTES);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&route_screen_kernel<true>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, CfgScreen::SMEM_BYTES);
}

}  // namespace moin
