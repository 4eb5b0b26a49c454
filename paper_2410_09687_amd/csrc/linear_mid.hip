// Prefill main kernels for calls of few tiles, and for contraction lengths that are not whole blocks (Section 3.2:
// y = W x + W_b (W_a x), one adapter per sequence).
//
// The products of linear_stream.hip, k-step for k-step in the same order, so that its results are the same bits, on
// 128 x 128 tiles: one per workgroup, four waves of 64 x 64 each, the hardware dealing the tiles out.
//  * What bounds it: LDS.  A block of 64 contraction steps takes 512 cycles of the matrix cores, 768 of LDS at its peak
//    (64 KB read by the waves, 32 KB written by the loads) and 600 of the path from L2 (55 bytes a cycle when an
//    instruction takes 128 bytes of each row); measured 1000-1100.  A 256 x 256 tile moves half of that per product, so
//    this kernel is for where too few of those tiles exist to fill the chip.
//  * Up to a tile per compute unit: four stages, three blocks in flight; beyond, two workgroups share a unit, two stages
//    each, and hide each other's waits, starts and epilogues.
//  * Rows may end anywhere (d_in and r any multiple of 8): in a row's last block the lanes past its end fetch zeros.
// Us of the kernel, 256 x 256 tiles / these: 1536 tokens 2048 -> 2048 43 / 20, 5632 -> 2048 96 / 41; 2560 tokens 43 / 29 and 97 /
// 66; 4096 tokens 45 / 34; 16 384 tokens 2048 -> 256 41 / 29; 8192 2048 -> 256 40 / 18.
#include <algorithm>
#include <type_traits>

#include "gemm_core.h"
#include "kernels.h"
#include "stream_epilogue.h"
#include "stream_tile.h"

namespace moin {

namespace mid {

using stream::BK;
using stream::ROWB;
constexpr int NW = 4, NT = NW * 64;

// BT_: tile edge, both ways
template <int BT_>
struct Shape {
    static constexpr int BT = BT_;
    static constexpr int FP = BT / 32, FQ = BT / 32;   // 16 x 16 accumulators per wave: half of the outputs x half of the tokens
    static constexpr int SUB = TILE_M / BT;            // tiles per plan tile
    static constexpr int P_BYTES = BT * ROWB, STAGE_BYTES = 2 * P_BYTES;
    static constexpr int LOADS = FP + FQ;              // requests of a wave per block, 8 rows each
    static constexpr int SCR_BYTES = 16 * FP * 16 * 4; // epilogue scratch of a wave: 16 tokens x its outputs, fp32
    static_assert(NW * SCR_BYTES <= 2 * STAGE_BYTES, "the scratch takes the stages' place");
};
constexpr int BT = 128, SUB = TILE_M / BT;
static_assert(SUB == 2, "HalfTiles");

// what the lanes past an operand row's end fetch
__device__ __align__(16) const unsigned int zero16[4] = {0, 0, 0, 0};

}  // namespace mid

template <int NS, bool Y_F32, bool RAGGED, int BT>
__device__ __forceinline__ void mid_tile(const stream::Params &p)
{
    using namespace mid;
    using S = Shape<BT>;
    constexpr int FP = S::FP, FQ = S::FQ, P_BYTES = S::P_BYTES, STAGE_BYTES = S::STAGE_BYTES, LOADS = S::LOADS, SCR_BYTES = S::SCR_BYTES;
    extern __shared__ __align__(16) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = uniform(threadIdx.x >> 6);
    const int wp = wave >> 1, wq = wave & 1;

    const std::conditional_t<S::SUB == 2, HalfTiles, QuarterTiles> parts(p.tile_rows, p.n_tiles, p.max_tiles);
    const int ntm = parts.count;
    const int id = xcd_band_id(blockIdx.x, ntm * p.n_tiles_n);
    if (id < 0) return;
    const int tm = p.by_columns ? id % ntm : id / p.n_tiles_n;
    const int tn = p.by_columns ? id / ntm : id % p.n_tiles_n;
    const stream::Tile t = stream::load_tile<BT, BT>(p, parts.find(tm), tn);
    if (t.q_rows <= 0) return;

    const int nkb0 = (p.d_in + BK - 1) / BK;
    const uint32_t ldx = (uint32_t)p.d_in * 2u, ldu = (uint32_t)p.ldu * 2u, ldb = (uint32_t)p.r * 2u;
    // Requests: number n of a wave fills 8 rows of an operand tile (the outputs' first); the lane fetches logical chunk
    // (lane % 8) ^ swz(row), swz(row) = (row >> 1) & 7.
    const uint32_t c16a = (((uint32_t)lane & 7) ^ ((uint32_t)lane >> 4)) * 16, c16b = c16a ^ 64u;   // even, odd
    uint32_t rowc[LOADS];
#pragma unroll
    for (int n = 0; n < LOADS; ++n) {
        const bool q = n >= FP;
        const uint32_t row = (uint32_t)((wave * FP + (n & (FP - 1))) * 8) + ((uint32_t)lane >> 3);
        rowc[n] = min(row, (uint32_t)((q ? t.q_rows : t.p_rows) - 1));
    }
    struct Fetch {
        const char *pp, *pq;
        uint32_t ldp, ldq, endp, endq;   // pitches; bytes of a row that are left at the block's start
    };
    auto fetch_of = [&](int b) __attribute__((always_inline)) {
        Fetch f;
        const bool base = b < nkb0;
        const int jb = b - nkb0;
        const bool hi = jb < t.nkb1;
        const int kb = base ? b : (hi ? jb : jb - t.nkb1);
        f.pq = (base ? t.q0 : (hi ? t.uh : t.ul)) + kb * ROWB;
        f.pp = (base ? t.p0 : t.be) + kb * ROWB;
        f.ldq = base ? ldx : ldu;
        f.ldp = base ? ldx : ldb;
        f.endq = f.ldq - (uint32_t)kb * ROWB;
        f.endp = f.ldp - (uint32_t)kb * ROWB;
        return f;
    };
    auto issue_one = [&](const Fetch &f, char *stage, int n) __attribute__((always_inline)) {
        const bool q = n >= FP;
        const int j = n & (FP - 1);
        const uint32_t c = (j & 1) ? c16b : c16a;
        const char *src = (q ? f.pq : f.pp) + (__umul24(rowc[n], q ? f.ldq : f.ldp) + c);
        if constexpr (RAGGED) src = c < (q ? f.endq : f.endp) ? src : reinterpret_cast<const char *>(zero16);
        __builtin_amdgcn_global_load_lds(MOIN_GPTR(src), MOIN_LPTR(stage + (q ? P_BYTES : 0) + (wave * FP + j) * 1024), 16, 0, 0);
    };

    // Fragments and MFMAs as in linear_stream.hip: row lane%16 of a 16-row block, k-step 1 at k-step 0's address ^ 64.
    const int lo0 = ((lane & 15) * ROWB) | ((((lane >> 4) ^ ((lane & 15) >> 1)) & 7) * 16);
    const int lo1 = lo0 ^ 64;
    const int baseP = wp * (FP * 16) * ROWB, baseQ = P_BYTES + wq * (FQ * 16) * ROWB;
    bf16x8_t fr[2][FP + FQ];
    auto read_one = [&](const char *stage, int lo_, int set, int n) __attribute__((always_inline)) {
        const int base_ = n < FP ? baseP + n * 16 * ROWB : baseQ + (n - FP) * 16 * ROWB;
        fr[set][n] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(stage + base_ + lo_));
    };
    auto frag_at = [](int k) { return k == 0 ? 0 : (k <= FQ ? FP + k - 1 : k - FQ); };
    f32x4_t acc[FP][FQ];
    auto mfma = [&](int set, int i, int j) __attribute__((always_inline)) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(fr[set][i]), "v"(fr[set][FP + j]));
    };
    auto mfma_first = [&](int i, int j) __attribute__((always_inline)) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc[i][j]) : "v"(fr[0][i]), "v"(fr[0][FP + j]));
    };

    const int total = t.total;
    constexpr int M = FP * FQ, R = FP + FQ;
    static_assert(M >= R, "a gap for every read and every request, or for the two together");
    constexpr int GAP = M >= 2 * R ? 2 : 1;   // MFMAs per read (and request) of the second k-step
    // One block: k-step 0 with the reads of k-step 1, the barrier, k-step 1 with the reads of the next block's k-step 0
    // and (MORE) the requests of the block NS ahead into the stage that is now free.
    auto body = [&](int b, char *st_cur, const char *st_nxt, auto first_tag, auto more_tag) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_tag)::value, MORE = decltype(more_tag)::value;
        Fetch f;
        if constexpr (MORE) f = fetch_of(b + NS);
#pragma unroll
        for (int n = 0; n < M; ++n) {
            if constexpr (FIRST) mfma_first(n / FQ, n % FQ);
            else mfma(0, n / FQ, n % FQ);
            if (n < R) {
                read_one(st_cur, lo1, 1, frag_at(n));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MORE) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * LOADS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int n = 0; n < M; ++n) {
            mfma(1, n / FQ, n % FQ);
            if (n % GAP == 0 && n / GAP < R) {
                read_one(st_nxt, lo0, 0, frag_at(n / GAP));
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (MORE)
                if (n % GAP == GAP - 1 && n / GAP < R) {
                    issue_one(f, st_cur, n / GAP);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        __builtin_amdgcn_sched_barrier(0);
    };

#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const Fetch f = fetch_of(min(s, total - 1));
#pragma unroll
        for (int n = 0; n < LOADS; ++n) issue_one(f, smem + s * STAGE_BYTES, n);
    }
    wait_vm_then_barrier<(NS - 1) * LOADS>();
#pragma unroll
    for (int n = 0; n < R; ++n) read_one(smem, lo0, 0, n);
    int st = 0;   // stage of block b
    auto next_of = [](int s) { return s + 1 == NS ? 0 : s + 1; };
    auto one = [&](int b, auto first_tag) __attribute__((always_inline)) {
        const int nx = next_of(st);
        char *cur = smem + st * STAGE_BYTES;
        const char *nxt = smem + nx * STAGE_BYTES;
        if (b + NS < total) body(b, cur, nxt, first_tag, std::true_type{});
        else body(b, cur, nxt, first_tag, std::false_type{});   // (the last block reads stale bytes that nothing uses)
        st = nx;
    };
    one(0, std::true_type{});
    int b = 1;
    for (; b + NS < total; ++b) {
        const int nx = next_of(st);
        body(b, smem + st * STAGE_BYTES, smem + nx * STAGE_BYTES, std::false_type{}, std::true_type{});
        st = nx;
    }
    for (; b < total; ++b) {
        const int nx = next_of(st);
        body(b, smem + st * STAGE_BYTES, smem + nx * STAGE_BYTES, std::false_type{}, std::false_type{});
        st = nx;
    }
    // Every wave has passed the last block's barrier with its fragments in registers and no request in flight, but the
    // stale reads of the last half block may still be under way where another wave's scratch will lie.
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // Epilogue, as in linear_stream.hip with half the outputs a wave (one function for both cost that kernel 0.5 %: its registers
    // are dealt out anew): a lane holds, per accumulator (i, j), token 16 j + lane%16 and outputs 16 i + 4 (lane/16) + 0..3; blocks of
    // 16 tokens are regrouped through the wave's scratch into whole lines of a token's row.
    {
        char *scr = smem + wave * SCR_BYTES;
        const int t16 = lane & 15, kg = lane >> 4;
        constexpr int EB = Y_F32 ? 4 : 2;
        constexpr int SLOT = 4 * EB;                // four outputs
        constexpr int ROW = FP * 16 * EB;           // a token's outputs
        constexpr int SLOTS = FP * 4;
        constexpr int CPR = ROW / 16;
        constexpr int SPC = 16 / SLOT;
        constexpr int NPS = 16 * CPR / 64;
        constexpr int TPP = 64 / CPR;
        const int tl = lane / CPR, ch = lane % CPR;
        const int n = wp * (FP * 16) + ch * (16 / EB);
        const bool n_ok = n < t.p_rows;             // d_out % 8 == 0: a chunk is all in or all out
        const uint32_t ldy = (uint32_t)t.d_out * EB;
        char *ybase = t.y + (int64_t)(t.row0 + wq * (FQ * 16)) * ldy + (int64_t)t.n0 * EB;
        const uint32_t voff = (uint32_t)tl * ldy + (uint32_t)n * EB;
        const int m_lane = wq * (FQ * 16) + tl;
#pragma unroll
        for (int j = 0; j < FQ; ++j) {
#pragma unroll
            for (int i = 0; i < FP; ++i) {
                const int slot_ = (i * 4 + kg) ^ ((2 * t16) & (SLOTS - 1));
                f32x4_t a;
#pragma unroll
                for (int e = 0; e < 4; ++e) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(a[e]) : "a"(acc[i][j][e]));
                if constexpr (Y_F32)
                    *reinterpret_cast<f32x4_t *>(scr + t16 * ROW + slot_ * SLOT) = a;
                else
                    *reinterpret_cast<uint2 *>(scr + t16 * ROW + slot_ * SLOT) =
                        make_uint2(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
            }
            lds_order();
            auto rd = [&](int ps) {
                const int tt = ps * TPP + tl;
                return *reinterpret_cast<const uint4 *>(scr + tt * ROW + ((ch * SPC) ^ ((2 * tt) & (SLOTS - 1))) * SLOT);
            };
            auto st_ = [&](int ps, const uint4 &v) {
                const int m = m_lane + j * 16 + ps * TPP;
                if (n_ok && m < t.q_rows)
                    *reinterpret_cast<uint4 *>(ybase + (uint32_t)(j * 16 + ps * TPP) * ldy + voff) = v;
            };
#pragma unroll
            for (int ps = 0; ps < NPS; ps += 2) {
                if constexpr (NPS == 1) {
                    st_(ps, rd(ps));
                } else {
                    const uint4 v0 = rd(ps), v1 = rd(ps + 1);
                    st_(ps, v0), st_(ps + 1, v1);
                }
            }
            lds_order();
        }
    }
}

template <int NS, bool Y_F32, bool RAGGED>
__global__ __launch_bounds__(mid::NT, NS == 2 ? 2 : 1) void linear_mid_kernel(stream::Params p)
{
    mid_tile<NS, Y_F32, RAGGED, mid::BT>(p);
}

// The same on 64 x 64 tiles, one per compute unit, eight stages: half the bytes through LDS per block and more blocks on
// their way, for calls of so few tiles that most of the chip would stand idle under the larger ones.  Us of the kernel,
// 128 x 128 / these: 500 tokens 2048 -> 2048 20 / 14, 330 2048 -> 2048, 256, 256 20 / 14, 4000 2048 -> 256 19 / 14, 640 1024 -> 1416
// 14 / 10, 1200 256 -> 256 9 / 8.  Beyond a tile per unit, 640 2048 -> 2048, 20 / 22.
constexpr int FINE_BT = 64, FINE_NS = 8;
template <bool Y_F32, bool RAGGED>
__global__ __launch_bounds__(mid::NT, 1) void linear_fine_kernel(stream::Params p)
{
    mid_tile<FINE_NS, Y_F32, RAGGED, FINE_BT>(p);
}

// The kernel for NS stages of BT x BT tiles.
template <int NS, int BT>
static auto mid_kernel(bool y_f32, bool ragged)
{
    if constexpr (BT == FINE_BT)
        return y_f32 ? (ragged ? &linear_fine_kernel<true, true> : &linear_fine_kernel<true, false>)
                     : (ragged ? &linear_fine_kernel<false, true> : &linear_fine_kernel<false, false>);
    else
        return y_f32 ? (ragged ? &linear_mid_kernel<NS, true, true> : &linear_mid_kernel<NS, true, false>)
                     : (ragged ? &linear_mid_kernel<NS, false, true> : &linear_mid_kernel<NS, false, false>);
}
template <int NS, int BT>
static hipError_t allow_lds_all()
{
    hipError_t e = hipSuccess;
    for (int v = 0; v < 4 && e == hipSuccess; ++v)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(mid_kernel<NS, BT>(v & 1, v & 2)),
                                hipFuncAttributeMaxDynamicSharedMemorySize, NS * mid::Shape<BT>::STAGE_BYTES);
    return e;
}

hipError_t prepare_mid_kernels()
{
    hipError_t e = allow_lds_all<2, mid::BT>();
    if (e == hipSuccess) e = allow_lds_all<4, mid::BT>();
    return e == hipSuccess ? allow_lds_all<FINE_NS, FINE_BT>() : e;
}

static int64_t mid_tiles(const PlanView &pv, const LinearArgs *a, int n, int bt = mid::BT)
{
    int64_t tn = 0;
    for (int i = 0; i < n; ++i) tn += (a[i].d_out + bt - 1) / bt;
    return host_tiles(pv, bt) * tn;
}

// Up to the tiles that the chip holds at a time, for each round that the 256 x 256 tiles need (two of these tiles per unit and
// round): with full row tiles, four of these in a large one, that is the first round's line alone, but where sequences end
// in the first half of a row tile, or a last round would be nearly empty, it lies further out.
// Us of the kernel, the streaming kernel's 256 x 256 tiles / these: 2048 -> 2048 448 tiles 42 / 31, 512 45 /
// 34, 544 45 / 52, 768 47 / 56, 1024 55 / 64 (one round of the larger tiles until then); beyond their first round 1152 89 / 84,
// 1280 90 / 87, but 1280 with 5632 outputs a call 106 / 113, so the line stays here; 5632 -> 2048 512 tiles 100 / 81,
// 544 101 / 132; 2048 -> 2048, 256, 256 480 tiles 46 / 33, 560 48 / 52; 528 tiles 2048 -> 5632 47 / 52.  Uneven sequences can
// make more tiles than the host takes them to: 16 of 60 to 430 tokens 560 instead of 512, 46 / 53 (were the line lower, as
// many even ones would lose 11).  Half-empty row tiles: 2048 -> 2048 64 sequences of 128 tokens (512 large tiles, 1024 of
// these) 109 / 71, 96 of 128 160 / 106, 20 of 300 (320, 960) 94 / 66; 2048 -> 11264 8 of 112 98 / 58, 32 of 112 305 / 198, 64 of
// 128 599 / 517, 4 of 300 (352, 1056: beyond the line) 98 / 85; 5632 -> 2048 64 of 128 244 / 158, 20 of 300 214 / 154; just
// beyond the line about equal (32 of 300 109 / 101, 24 of 512 99 / 102), further out the large ones win (32 of 512 112 / 133).
// Against tiles that go through registers (rows that are not whole blocks), us of a call: 1000 -> 2048 256 tiles 50 / 30,
// 1024 59 / 62, 1416 -> 5632 at 11264 654 / 776; half-empty ones 1000 -> 2048 40 sequences of 80 tokens 83 / 51, 64 of 64 at
// rank 64 92 / 59, 128 of 64 169 / 100; 1000 -> 5632 12 of 96 85 / 49, 64 of 80 246 / 139; sequences of 129 to 1000
// tokens the same within what runs differ.
bool mid_kernel_pays(const PlanView &pv, const LinearArgs *a, int n, int n_cus)
{
    int64_t tn = 0;
    for (int i = 0; i < n; ++i) tn += (a[i].d_out + TILE_M - 1) / TILE_M;
    return mid_tiles(pv, a, n) <= 2 * n_cus * tile_rounds(pv, tn, n_cus);
}

template <int NS, int BT>
static hipError_t launch_mid(const PlanView &pv, const LinearArgs *a, int n, hipStream_t stream_)
{
    using S = mid::Shape<BT>;
    stream::Params p;
    const int tn = stream::fill_params(&p, pv, a, n, BT);
    // the larger operand's rows are dealt out over the XCDs, the smaller one is read by all of them
    p.by_columns = (int64_t)tn * BT > pv.T;
    const int64_t work = (int64_t)pv.max_tiles * S::SUB * tn;
    if (work > 0x7ffffff0LL) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)((work + 7) / 8 * 8);
    const bool ragged = p.r % mid::BK != 0 || p.d_in % mid::BK != 0;
    hipLaunchKernelGGL((mid_kernel<NS, BT>(p.y_f32, ragged)), dim3(grid), dim3(mid::NT), NS * S::STAGE_BYTES, stream_, p);
    return hipGetLastError();
}

hipError_t launch_linear_mid(const PlanView &pv, const LinearArgs *a, int n, int n_cus, hipStream_t stream_)
{
    if (n < 1 || n > MAX_SHARED_X) return hipErrorInvalidValue;
    if (pv.max_tiles <= QuarterTiles::MAX && mid_tiles(pv, a, n, FINE_BT) <= n_cus) return launch_mid<FINE_NS, FINE_BT>(pv, a, n, stream_);
    // (Us of the kernel, four stages / two: 240 tiles 20 / 25, 256 22 / 26, 268 37 / 29, 320 36 / 30.)
    if (mid_tiles(pv, a, n) <= n_cus) return launch_mid<4, mid::BT>(pv, a, n, stream_);
    return launch_mid<2, mid::BT>(pv, a, n, stream_);
}

}  // namespace moin
