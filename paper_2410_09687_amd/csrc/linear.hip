// Prefill path of the routed LoRA linear layer (Section 3.2:
// y = W x + W_b (W_a x), one adapter per sequence).
//
//   shrink : u = scale * x A_e^T, written as a bf16 pair (u_hi + u_lo) so the
//            expand product sees ~16 significant bits of u.
//   linear : y = x W^T + u_hi B_e^T + u_lo B_e^T  -- the adapter term is simply
//            2r more contraction steps appended to the base GEMM of the same
//            output tile, so y is written once, from one fp32 accumulator.
// Tiles come from the plan: no tile spans two sequences, hence one adapter per
// tile.  The same linear kernel, in a smaller tile shape and over a regular
// grid of tiles, is the decode path's base GEMM; there the contraction range
// may be cut into several parts, each writing its own fp32 partial result.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "gemm_core.h"
#include "kernels.h"
#include "linear_tile.h"

namespace moin {


struct ShrinkKParams {
    const char *x, *A_stack;
    char *u_hi, *u_lo;
    // projections that share x: column tile tn belongs to projection tn / tiles_per_proj
    // (A_stack / u_hi / u_lo above are then those of projection 0)
    int n_proj, tiles_per_proj;
    const char *A_more[MAX_SHARED_X - 1];
    char *uh_more[MAX_SHARED_X - 1], *ul_more[MAX_SHARED_X - 1];
    const int *tile_row0, *tile_rows, *tile_expert, *tile_rank, *n_tiles;
    int d_in, r, ldu;
    int n_tiles_n;
    float scale;
    int act;
    // QUANT only: MXFP8 codes [T, d_in] and scale bytes [d_in / 128, T, 4] of x
    char *xq, *xs;
    int64_t T;
};

// MXFP8 quantisation of one thread's 8 consecutive values of x (w: four words of
// two bf16 each) whose block of 32 lies in four neighbouring lanes: the block's
// scale byte E = max(0, exponent field of the largest magnitude - 8), 127 for a
// block of zeros; elements = value / 2^(E - 127), clamped to +-448, rounded to
// nearest even ("Future Works", quantising the base model; OCP Microscaling
// format).  Returns the 8 codes; E through `scale_byte`.
// Magnitudes are compared two at a time, neighbours exchange through DPP and not through LDS, the clamp is one
// instruction.  With the walk's loads counted exactly (pipelined_blocks_deep) the pass takes, 18 700 x 2048 at rank 64,
// 48 -> 42 us, x 5632 124 -> 108; 64-row tiles (48 us) and stores without a condition (43) are no better.
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_FROM_PLUS4 = 0x104;   // quad_perm [1,0,3,2], [2,3,0,1]; row_shl 4
__device__ __forceinline__ uint2 mx_quantize8(const uint4 &v, int &scale_byte)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    u16x2_t m2 = __builtin_bit_cast(u16x2_t, w[0] & 0x7FFF7FFFu);
#pragma unroll
    for (int i = 1; i < 4; ++i) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(u16x2_t, w[i] & 0x7FFF7FFFu));
    int m = max((int)m2[0], (int)m2[1]);
    m = max(m, dpp_move<DPP_XOR1>(m));
    m = max(m, dpp_move<DPP_XOR2>(m));
    const int E = m == 0 ? 127 : max(0, (m >> 7) - 8);
    const float inv = bits_f32((uint32_t)(254 - E) << 23);   // 2^(127 - E)
    float f[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __builtin_amdgcn_fmed3f(bits_f32(w[i] << 16) * inv, -448.f, 448.f);
        f[2 * i + 1] = __builtin_amdgcn_fmed3f(bits_f32(w[i] & 0xFFFF0000u) * inv, -448.f, 448.f);
    }
    int lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[0], f[1], 0, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[2], f[3], lo, true);
    int hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[4], f[5], 0, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[6], f[7], hi, true);
    scale_byte = E;
    return make_uint2((uint32_t)lo, (uint32_t)hi);
}

// u for 4 consecutive columns, the first `left` of which exist (the others are zeros), as a bf16 pair.
__device__ __forceinline__ void u_pair(const f32x4_t &v, int left, int act, float s, uint2 &hi, uint2 &lo)
{
    uint32_t h[4], l[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float f = q < left ? adapter_act(v[q], act) * s : 0.f;
        h[q] = f32_to_bf16_bits(f);
        l[q] = f32_to_bf16_bits(f - bf16_bits_to_f32(h[q]));
    }
    hi = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
    lo = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
}

// QUANT (register-staged tile shapes with BK = 64, d_in a multiple of 128): the
// pass over x also writes x in MXFP8 for the quantised-base layer, so that x
// comes from HBM once for both.  The workgroups of the first column tile do it,
// also for tiles without an adapter, which the plain shrink skips.
template <class C, bool QUANT = false>
__global__ __launch_bounds__(C::NT) void shrink_kernel(ShrinkKParams p)
{
    extern __shared__ __align__(16) char smem[];
    constexpr int SUB = TILE_M / C::BM;
    const int ntm = uniform(*p.n_tiles) * SUB;
    // neighbouring sub-tiles share A_e: keep them on one XCD so that its L2
    // fetches each adapter slab from HBM once
    const int id = xcd_band_id(blockIdx.x, ntm * p.n_tiles_n);
    if (id < 0) return;
    const int tm = uniform(id / p.n_tiles_n), tn = uniform(id % p.n_tiles_n);
    const int t = tm / SUB, sub = tm % SUB;
    const int e = uniform(p.tile_expert[t]);
    int rows = uniform(p.tile_rows[t]) - sub * C::BM;
    const bool quant = QUANT && tn == 0;
    if (rows <= 0 || (e < 0 && !quant)) return;
    rows = min(rows, C::BM);
    const int row0 = uniform(p.tile_row0[t]) + sub * C::BM;
    const int proj = tn / p.tiles_per_proj;
    const int n0 = (tn - proj * p.tiles_per_proj) * C::BN;
    const char *A_stack = p.A_stack;
    char *u_hi = p.u_hi, *u_lo = p.u_lo;
#pragma unroll
    for (int i = 1; i < MAX_SHARED_X; ++i)
        if (proj == i) {   // (selected one by one: indexing the arrays would put the parameters in scratch)
            A_stack = p.A_more[i - 1];
            u_hi = p.uh_more[i - 1];
            u_lo = p.ul_more[i - 1];
        }
    // the expert's own rank: rows of A_e beyond it do not exist; the main kernel
    // reads u in blocks of 64 columns, so the rest of the last block is written as zeros
    const int re = e < 0 ? 0 : min(p.r, uniform(p.tile_rank[t]));
    const int r_read = min(p.ldu, (re + 63) & ~63);
    const bool shrink = n0 < r_read;
    if (!shrink && !quant) return;
    const int ncols = max(1, min(C::BN, re - n0));      // rows of A_e to fetch (at least one, in bounds)
    const int ncols_out = min(C::BN, r_read - n0);      // columns of u to write

    const uint32_t ldx = (uint32_t)p.d_in * 2u;
    const char *xa = p.x + (int64_t)row0 * ldx;
    // (a walk for the quantiser alone puts x in A_e's place: valid addresses, unused products)
    const char *ae = shrink ? A_stack + ((int64_t)e * p.r + n0) * ldx : xa;
    const int nkb = (p.d_in + C::BK - 1) / C::BK;

    // Workgroups that start together would all ask for the same 128 bytes of their rows, one row
    // pitch (4 KB and up) apart from the next: requests that pile up on a few memory channels.  Each
    // 256-row tile therefore starts its walk over the contraction at another block and wraps round
    // (the sub-tiles of a tile, and the projections that share x, keep one phase so that they meet
    // in L2): 88 -> 70 us for a 65536 x 2048 pass at rank 128.  The phase comes from the tile's
    // position in the batch, not from its place in the by-expert order, and is the same in every
    // variant of this kernel and in shrink_patch_kernel, so that a row's sum depends neither on how the
    // experts are numbered nor on which of them ran.
    const int k_first = (int)(((uint32_t)(row0 - sub * C::BM) / (uint32_t)TILE_M * 5u) % (uint32_t)nkb);
    auto block_of = [=](int it) __attribute__((always_inline)) {
        const int kb = it + k_first;
        return kb >= nkb ? kb - nkb : kb;
    };

    typename C::Acc acc;
    C::zero(acc);
    if constexpr (C::IS_DMA) {
        const auto la = C::template make_lanes<C::A_I>(rows);
        const auto lb = C::template make_lanes<C::B_I>(ncols);
        auto issue = [=](int it, char *stage) __attribute__((always_inline)) {
            C::issue(stage, xa, ldx, la, ae, ldx, lb, (uint32_t)block_of(it) * (C::BK * 2));
        };
        dma_pipelined_blocks<C>(smem, nkb, issue, acc, [](int) {});
    } else {
        const auto vx = C::template make_view<C::A_CH>(xa, ldx, rows);
        const auto va = C::template make_view<C::B_CH>(ae, ldx, shrink ? ncols : rows);
        auto issue = [=](int it, typename C::Stage &g) __attribute__((always_inline)) {
            C::load_stage(g, vx, va, (uint32_t)block_of(it) * (C::BK * 2), ldx);
        };
        if constexpr (C::PF > 1) {
            static_assert(!QUANT || C::BK == 64, "a block of 32 values in four neighbouring lanes, two per row");
            const int qrow = threadIdx.x / C::KCH, kc = threadIdx.x % C::KCH;
            auto walk = [&](auto quantise) __attribute__((always_inline)) {
                pipelined_blocks_deep<C, C::PF>(smem, nkb, issue, acc, [&](int it, const typename C::Stage &g)
                                                                           __attribute__((always_inline)) {
                    if constexpr (decltype(quantise)::value) {
#pragma unroll
                        for (int i = 0; i < C::A_CH; ++i) {
                            int E;
                            const uint2 codes = mx_quantize8(g.a[i], E);
                            // the two scale bytes of a row's 64 values, into the row's first thread
                            const uint32_t pair = (uint32_t)E | ((uint32_t)dpp_move<DPP_FROM_PLUS4>(E) << 8);
                            const int row = qrow + i * C::RPP;
                            if (row < rows) {
                                const int k0 = block_of(it) * 64;
                                *reinterpret_cast<uint2 *>(p.xq + (int64_t)(row0 + row) * p.d_in + k0 + kc * 8) = codes;
                                if (kc == 0)
                                    *reinterpret_cast<uint16_t *>(p.xs + ((int64_t)(k0 >> 7) * p.T + row0 + row) * 4 +
                                                                  ((k0 >> 5) & 3)) = (uint16_t)pair;
                            }
                        }
                    }
                });
            };
            if (quant) walk(std::integral_constant<bool, QUANT>{});
            else walk(std::false_type{});
        } else {
            pipelined_blocks<C>(smem, nkb, issue, acc);
        }
    }
    if (!shrink) return;

    const int64_t ldu = (int64_t)p.ldu * 2;
    char *uh = u_hi + (int64_t)row0 * ldu;
    char *ul = u_lo + (int64_t)row0 * ldu;
    const float s = p.scale;
    const int act = p.act;
    C::epilogue(smem, acc, [&](int row, int col, float(&v)[8]) {
        if (row >= rows || col >= ncols_out) return;
        uint2 h0, l0, h1, l1;
        u_pair(f32x4_t{v[0], v[1], v[2], v[3]}, re - n0 - col, act, s, h0, l0);
        u_pair(f32x4_t{v[4], v[5], v[6], v[7]}, re - n0 - col - 4, act, s, h1, l1);
        const int64_t off = (int64_t)row * ldu + (int64_t)(n0 + col) * 2;
        *reinterpret_cast<uint4 *>(uh + off) = make_uint4(h0.x, h0.y, h1.x, h1.y);
        *reinterpret_cast<uint4 *>(ul + off) = make_uint4(l0.x, l0.y, l1.x, l1.y);
    });
}

template <int... K, class F>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, K...>, F f)
{
    (f(std::integral_constant<int, K>{}), ...);
}

// x in MXFP8: a lane's 8 values of row `row` (of `rows`, from row0 on) and of the block of 64 from k0 on, lanes 0..7 holding the
// first of a wave's eight rows.
__device__ __forceinline__ void quantise_group(const ShrinkKParams &p, const uint4 &v, int row0, int row, int rows, int k0)
{
    const int c = threadIdx.x & 7;
    int E;
    const uint2 codes = mx_quantize8(v, E);
    // the two scale bytes of a row's 64 values, into the row's first lane
    const uint32_t pair = (uint32_t)E | ((uint32_t)dpp_move<DPP_FROM_PLUS4>(E) << 8);
    if (row < rows) {
        *reinterpret_cast<uint2 *>(p.xq + (int64_t)(row0 + row) * p.d_in + k0 + c * 8) = codes;
        if (c == 0)
            *reinterpret_cast<uint16_t *>(p.xs + ((int64_t)(k0 >> 7) * p.T + row0 + row) * 4 + ((k0 >> 5) & 3)) = (uint16_t)pair;
    }
}

// x in MXFP8: blocks first, first + step, ... of `rows` (1 to 8 RG) rows, counted from block k_first on, by one wave.  PF - 1
// blocks' loads are under way while one is worked on; 8 lanes hold a row's 64 values.
template <int RG, int PF>
__device__ __forceinline__ void quantise_rows(const ShrinkKParams &p, int row0, int rows, int k_first, int first, int step)
{
    const int lane = threadIdx.x & 63, c = lane & 7, nkb = p.d_in / 64;
    const int n = (nkb - first + step - 1) / step;
    if (n <= 0) return;
    auto block_of = [=](int i) __attribute__((always_inline)) {
        const int kb = first + i * step + k_first;
        return kb >= nkb ? kb - nkb : kb;
    };
    const char *xa = p.x + (int64_t)row0 * p.d_in * 2;
    uint32_t off[RG];
#pragma unroll
    for (int j = 0; j < RG; ++j) off[j] = (uint32_t)min(j * 8 + (lane >> 3), rows - 1) * ((uint32_t)p.d_in * 2u) + (uint32_t)c * 16u;
    uint4 v[PF][RG];
    auto load = [&](int i, uint4(&g)[RG]) __attribute__((always_inline)) {
        const uint32_t at = (uint32_t)block_of(min(i, n - 1)) * 128u;   // (past the end the last block once more: no branch)
#pragma unroll
        for (int j = 0; j < RG; ++j) g[j] = *reinterpret_cast<const uint4 *>(xa + (off[j] + at));
    };
    auto work = [&](int i, const uint4(&g)[RG]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < RG; ++j) quantise_group(p, g[j], row0, j * 8 + (lane >> 3), rows, block_of(i) * 64);
    };
#pragma unroll
    for (int u = 0; u < PF; ++u) load(u, v[u]);
    for (int i = 0; i < n; i += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            if (i + u < n) work(i + u, v[u]);
            load(i + u + PF, v[u]);
        }
    }
}

// The shrink of batches whose larger tiles do not fill the chip: the sums of the kernel above, product for product in the same
// order, so that a sequence's u is the same bits in a batch of any size.  Bound by the chain of a tile's blocks of 64 steps,
// which the tiles above work off at 0.35 us each, on as many compute units as there are tiles; and beyond some 5000 tokens by
// what the tiles fetch, x once for every tile of columns.  Here a wave holds 32 tokens x 16 or 32 columns, and the next
// block's fragments come to registers under the products of the present one: 0.12 and 0.16 us a block, the wave's own stream of
// requests, reads and products.  In the smallest batches a wave is a workgroup, with stages that nobody else waits for; in larger ones
// two or four share a tile of 64 tokens, and a barrier a block.  (16 columns, us by 5632 of 1890 tokens with adapters from HBM: six stages
// 18.2, eight 15.9, ten 17.1; tiles of several waves are no faster with six than with four.)
// With codes as well (QW): waves of their own make them, since a block's 32 x 64 values cost a wave 0.5 us.
// The rule below gives times.
template <int FN_, int WM_, int WN_, int NS_>
struct PatchCfg {
    static constexpr int FM = 2, FN = FN_, WM = WM_, WN = WN_, NW = WM * WN;
    static constexpr int BM = WM * FM * 16, BN = WN * FN * 16, BK = 64, ROWB = BK * 2;
    static constexpr int A_I = BM / 8, B_I = BN / 8, LPB = (A_I + B_I) / NW;   // requests per block, 8 rows each; of a wave
    static constexpr int STAGE_BYTES = (BM + BN) * ROWB;
    static constexpr int NS = NS_, SMEM_BYTES = NS * STAGE_BYTES;
    static_assert((A_I + B_I) % NW == 0 && (NS - 1) * LPB < 64 && NS % 2 == 0, "requests; vmcnt field; registers by parity");
};
using CfgPatch16 = PatchCfg<1, 1, 1, 8>;
using CfgPatch32 = PatchCfg<2, 2, 1, 4>;
using CfgPatch64 = PatchCfg<2, 2, 2, 4>;
using CfgPatchWide = PatchCfg<2, 1, 2, 4>;   // with codes at rank 64: x once, and twice as many tiles

// QW: further waves of each workgroup, which write x in MXFP8, also where there is no adapter: beside a single patch each its
// share of the row tile's blocks, from memory; beside several its share of every block's rows, from LDS.
template <class C, int QW>
__global__ __launch_bounds__(64 * (C::NW + QW)) void shrink_patch_kernel(ShrinkKParams p)
{
    extern __shared__ __align__(16) char smem[];
    constexpr int SUB = TILE_M / C::BM, FN = C::FN;
    const int ntm = uniform(*p.n_tiles) * SUB;
    const int id = xcd_band_id(blockIdx.x, ntm * p.n_tiles_n);
    if (id < 0) return;
    const int tm = uniform(id / p.n_tiles_n), tn = uniform(id % p.n_tiles_n);
    const int t = tm / SUB, sub = tm % SUB;
    const int rows = min(uniform(p.tile_rows[t]) - sub * C::BM, C::BM);
    if (rows <= 0) return;
    const int row0 = uniform(p.tile_row0[t]) + sub * C::BM;
    const int nkb = p.d_in / C::BK;
    const int k_first = (int)(((uint32_t)(row0 - sub * C::BM) / (uint32_t)TILE_M * 5u) % (uint32_t)nkb);
    const int wave = uniform(threadIdx.x >> 6);
    if (QW > 0 && C::NW == 1 && wave > 0) {
        quantise_rows<4, 3>(p, row0, rows, k_first, tn * QW + wave - 1, p.n_tiles_n * QW);
        return;
    }
    const int e = uniform(p.tile_expert[t]);
    const int re = e < 0 ? 0 : min(p.r, uniform(p.tile_rank[t]));
    const int r_read = min(p.ldu, (re + 63) & ~63);   // columns of u that are read: zeros from the rank on
    const int proj = tn / p.tiles_per_proj, tc = tn - proj * p.tiles_per_proj;
    const int n0 = tc * C::BN;
    // the columns to write: the tile's own, behind the last tile also what is left of a block of 64
    const int n_end = tc + 1 == p.tiles_per_proj ? r_read : min(r_read, n0 + C::BN);
    if constexpr (QW > 0 && C::NW > 1) {
        if (wave >= C::NW) {
            const int g0 = wave - C::NW + tc * QW, g_step = QW * p.tiles_per_proj;   // the wave's groups of eight rows
            if (n0 >= re) {   // (no products, nothing in LDS)
                for (int g = g0; g * 8 < rows; g += g_step) quantise_rows<1, 6>(p, row0 + g * 8, min(rows - g * 8, 8), k_first, 0, 1);
                return;
            }
            // Block it lies in its stage from the barrier of the turn before on (the first from the one ahead of the
            // turns) until that of its own turn: as many barriers as the product waves meet.
            const int l = threadIdx.x & 63;
            wait_vm_then_barrier<63>();
            for (int it = 0; it < nkb; ++it) {
                const char *st = smem + (it % C::NS) * C::STAGE_BYTES;
                const int kb = it + k_first, k0 = (kb >= nkb ? kb - nkb : kb) * C::BK;
                for (int g = g0; g < C::BM / 8; g += g_step) {
                    const int row = g * 8 + (l >> 3);
                    quantise_group(p, *reinterpret_cast<const uint4 *>(st + row * C::ROWB + (((l & 7) ^ ((row >> 1) & 7)) * 16)), row0, row, rows, k0);
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
            return;
        }
    }
    if (n0 >= n_end) return;
    const char *A_stack = p.A_stack;
    char *u_hi = p.u_hi, *u_lo = p.u_lo;
#pragma unroll
    for (int i = 1; i < MAX_SHARED_X; ++i)
        if (proj == i) {
            A_stack = p.A_more[i - 1];
            u_hi = p.uh_more[i - 1];
            u_lo = p.ul_more[i - 1];
        }

    const int lane = threadIdx.x & 63;
    const int wm = wave / C::WN, wn = wave % C::WN;
    f32x4_t acc[C::FM][FN];
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (n0 < re) {   // (else: zeros alone)
        const uint32_t ldx = (uint32_t)p.d_in * 2u;
        const char *xa = p.x + (int64_t)row0 * ldx;
        const char *ae = A_stack + ((int64_t)e * p.r + n0) * ldx;
        const int a_rows = min(C::BN, re - n0);
        // as in DmaCore: 8 rows of 128 bytes a request, 16-byte chunks XORed with swz(row) = (row >> 1) & 7; x's rows, then A's
        uint32_t off[C::LPB];
#pragma unroll
        for (int j = 0; j < C::LPB; ++j) {
            const int g = wave * C::LPB + j;
            const bool a = g < C::A_I;
            const int row = (a ? g : g - C::A_I) * 8 + (lane >> 3);
            const uint32_t c16 = (((uint32_t)lane & 7) ^ ((uint32_t)lane >> 4) ^ ((uint32_t)(g & 1) * 4u)) * 16;
            off[j] = (uint32_t)min(row, (a ? rows : a_rows) - 1) * ldx + c16;
        }
        auto kbyte_of = [&](int it) __attribute__((always_inline)) {
            const int kb = it + k_first;
            uint32_t k = (uint32_t)(kb >= nkb ? kb - nkb : kb) * C::ROWB;
            asm volatile("" : "+s"(k));   // (one addition per request; taken apart it becomes three)
            return k;
        };
        auto issue_one = [&](uint32_t kbyte, char *st, int j) __attribute__((always_inline)) {
            const int g = wave * C::LPB + j;
            __builtin_amdgcn_global_load_lds(MOIN_GPTR((g < C::A_I ? xa : ae) + (off[j] + kbyte)), MOIN_LPTR(st + g * 1024), 16, 0, 0);
        };
        auto stage = [&](int it) __attribute__((always_inline)) { return smem + (it % C::NS) * C::STAGE_BYTES; };
        // fragments: row lane % 16 of 16, the second half of a block at the first one's address ^ 64; of the tokens, then the columns
        const int lo = (lane & 15) * C::ROWB | ((((lane >> 4) ^ ((lane & 15) >> 1)) & 7) * 16);
        const int base_x = wm * (C::FM * 16) * C::ROWB, base_a = (C::BM + wn * (FN * 16)) * C::ROWB;
        constexpr int F = C::FM + FN, R = 2 * F, M = 2 * C::FM * FN;   // fragments of a half; reads and products of a block
        bf16x8_t fr[2][R];
        auto read_one = [&](const char *st, int set, int n) __attribute__((always_inline)) {
            const int f = n % F, at = f < C::FM ? base_x + f * 16 * C::ROWB : base_a + (f - C::FM) * 16 * C::ROWB;
            fr[set][n] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(st + at + (lo ^ (n / F * 64))));
        };
        auto product = [&](int set, int n) __attribute__((always_inline)) {
            const int ks = n / (M / 2), i = n % (M / 2) / FN, j = n % FN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[set][ks * F + C::FM + j], fr[set][ks * F + i], acc[i][j], 0, 0, 0);
        };
        // Block it, whose fragments are in registers behind the wait.  LEFT blocks beyond the next one may still be under way;
        // its stage, read out (by all waves, behind the barrier), takes block it + NS (MORE), the next block's fragments come to
        // the other registers (NEXT).
        auto turn = [&](int it, auto set_tag, auto left_tag, auto more_tag, auto next_tag) __attribute__((always_inline)) {
            constexpr int SET = decltype(set_tag)::value, LEFT = decltype(left_tag)::value;
            constexpr bool MORE = decltype(more_tag)::value, NEXT = decltype(next_tag)::value;
            if constexpr (C::NW == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LEFT * C::LPB) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LEFT * C::LPB) : "memory");
            const uint32_t kbyte = MORE ? kbyte_of(it + C::NS) : 0;
            char *cur = stage(it);
            const char *nxt = stage(it + 1);
#pragma unroll
            for (int n = 0; n < (M > R ? M : R); ++n) {
                if (n < M) product(SET, n);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (NEXT)
                    if (n < R) read_one(nxt, 1 - SET, n);
                if constexpr (MORE)
                    if (n < C::LPB) issue_one(kbyte, cur, n);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        using T_ = std::true_type;
        using F_ = std::false_type;
        using S0 = std::integral_constant<int, 0>;
        using S1 = std::integral_constant<int, 1>;
        using Full = std::integral_constant<int, C::NS - 2>;
        auto fetch = [&](int it) __attribute__((always_inline)) {
            const uint32_t kbyte = kbyte_of(it);
#pragma unroll
            for (int j = 0; j < C::LPB; ++j) issue_one(kbyte, stage(it), j);
        };
        auto landed = [](auto left_tag) __attribute__((always_inline)) {
            if constexpr (C::NW == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(left_tag)::value * C::LPB) : "memory");
            else wait_vm_then_barrier<decltype(left_tag)::value * C::LPB>();
        };
        auto read_block = [&](int it, int set) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < R; ++n) read_one(stage(it), set, n);
        };
        if (nkb >= C::NS) {
#pragma unroll
            for (int s = 0; s < C::NS; ++s) fetch(s);
            landed(std::integral_constant<int, C::NS - 1>{});
            const int more = nkb - C::NS;   // turns that fetch; the first of an odd number by itself, so that the last NS begin with set 0
            int it = 0;
            if (more & 1) {
                read_block(0, 1);
                turn(0, S1{}, Full{}, T_{}, T_{});
                it = 1;
            } else {
                read_block(0, 0);
            }
            for (; it < more; it += 2) {
                turn(it, S0{}, Full{}, T_{}, T_{});
                turn(it + 1, S1{}, Full{}, T_{}, T_{});
            }
            unrolled(std::make_integer_sequence<int, C::NS>{}, [&](auto k) __attribute__((always_inline)) {
                constexpr int K = decltype(k)::value;
                turn(it + K, std::integral_constant<int, (K & 1)>{}, std::integral_constant<int, (K + 2 < C::NS ? C::NS - 2 - K : 0)>{},
                     F_{}, std::integral_constant<bool, (K + 1 < C::NS)>{});
            });
        } else {
            for (int s = 0; s < nkb; ++s) fetch(s);
            landed(S0{});
            for (int it = 0; it < nkb; ++it) {
                read_block(it, 0);
                turn(it, S0{}, S0{}, F_{}, F_{});
            }
        }
    }

    // a lane holds, per accumulator (i, j), token 16 i + lane % 16 and columns 16 j + 4 (lane / 16) + 0..3
    const int64_t ldu = (int64_t)p.ldu * 2;
    const int n0w = n0 + wn * (FN * 16);
#pragma unroll
    for (int i = 0; i < C::FM; ++i) {
        const int row = wm * (C::FM * 16) + i * 16 + (lane & 15);
        if (row >= rows) continue;
        const int64_t at = (int64_t)(row0 + row) * ldu;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int col = n0w + j * 16 + 4 * (lane >> 4);
            if (col >= n_end) continue;
            uint2 hi, lo;
            u_pair(acc[i][j], re - col, p.act, p.scale, hi, lo);
            *reinterpret_cast<uint2 *>(u_hi + at + col * 2) = hi;
            *reinterpret_cast<uint2 *>(u_lo + at + col * 2) = lo;
        }
        if (wn + 1 == C::WN)
            for (int col = n0 + C::BN + 4 * (lane >> 4); col < n_end; col += 16) {
                *reinterpret_cast<uint2 *>(u_hi + at + col * 2) = make_uint2(0, 0);
                *reinterpret_cast<uint2 *>(u_lo + at + col * 2) = make_uint2(0, 0);
            }
    }
}

// Tile shapes.  The *Dma variants need the contraction length to be a multiple
// of BK = 64; the register-staged ones take any multiple of 8.  CfgMain is for
// contraction lengths the streaming kernel (linear_stream.hip) does not take, in calls of more tiles
// than linear_mid.hip takes.
using CfgMain = GemmCore<256, 256, 64, 4, 2>;        // 8 waves, wave patch 64 x 128
using CfgShrink = GemmCore<64, 64, 64, 2, 2>;        // 4 waves, wave patch 32 x 32
using CfgShrinkDma = DmaCore<64, 64, 64, 2, 2, 4>;
// ranks from 65 to 128: the whole rank in one tile, so x streams from HBM once
using CfgShrinkR128 = DmaCore<128, 128, 64, 2, 4, 2>;   // (two stages of 64 steps: 5632-deep rows 15 % faster than four of 32)
// the quantising variant: register-staged (the quantiser works on the registers on
// their way to LDS), the loads of four blocks in flight per thread
template <int BM, int BN, int BK, int WM, int WN, int PF_>
struct DeepCore : GemmCore<BM, BN, BK, WM, WN> {
    static constexpr int PF = PF_;
};
using CfgShrinkDeep = DeepCore<128, 128, 64, 2, 4, 4>;   // ranks 65..128
using CfgShrinkDeep64 = DeepCore<128, 64, 64, 4, 2, 4>;  // ranks up to 64, and above 128 in column tiles

template <class K>
static hipError_t allow_lds(K kern, int bytes)
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

hipError_t prepare_stream_kernel();
bool stream_kernel_fits(const LinearArgs &a);
hipError_t launch_linear_stream(const PlanView &pv, const LinearArgs &a, int n_cus, hipStream_t stream);
hipError_t launch_linear_stream_shared(const PlanView &pv, const LinearArgs *a, int n, int n_cus, hipStream_t stream);

hipError_t prepare_linear_kernels()
{
    hipError_t e;
    if ((e = prepare_stream_kernel()) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_patch_kernel<CfgPatch16, 0>, CfgPatch16::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_patch_kernel<CfgPatch32, 0>, CfgPatch32::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_patch_kernel<CfgPatch64, 0>, CfgPatch64::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_patch_kernel<CfgPatch16, 1>, CfgPatch16::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_patch_kernel<CfgPatchWide, 4>, CfgPatchWide::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_patch_kernel<CfgPatch64, 4>, CfgPatch64::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&linear_kernel<CfgMain>, CfgMain::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&linear_kernel<CfgThin>, CfgThin::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&linear_kernel<CfgDecodeBase>, CfgDecodeBase::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_kernel<CfgShrink>, CfgShrink::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_kernel<CfgShrinkR128>, CfgShrinkR128::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_kernel<CfgShrinkDma>, CfgShrinkDma::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_kernel<CfgShrinkDeep, true>, CfgShrinkDeep::SMEM_BYTES)) != hipSuccess) return e;
    return allow_lds(&shrink_kernel<CfgShrinkDeep64, true>, CfgShrinkDeep64::SMEM_BYTES);
}

static inline int round_up8(int v) { return (v + 7) & ~7; }

// Compute units of the current device (queried once per device).
int compute_units()
{
    static int cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

// xq / xs: the quantising variant's outputs
struct SharedX {
    int n;
    const void *const *A_stack;
    void *const *u_hi, *const *u_lo;
};

// Column tiles of bn; returns the number of workgroups with row tiles of bm (negative: too many).
static int64_t shrink_params(ShrinkKParams &p, const PlanView &pv, const LinearArgs &a, const SharedX *shared, void *xq,
                             void *xs, int bm, int bn)
{
    p.xq = (char *)xq; p.xs = (char *)xs; p.T = pv.T;
    p.x = (const char *)a.x; p.A_stack = (const char *)a.A_stack;
    p.u_hi = (char *)a.u_hi; p.u_lo = (char *)a.u_lo;
    p.tile_row0 = pv.tile_row0; p.tile_rows = pv.tile_rows; p.tile_expert = pv.tile_expert;
    p.tile_rank = pv.tile_rank;
    p.n_tiles = pv.n_tiles;
    p.d_in = a.d_in; p.r = a.r; p.ldu = a.ldu; p.scale = a.scale; p.act = a.act;
    p.tiles_per_proj = (a.r + bn - 1) / bn;
    p.n_proj = shared ? shared->n : 1;
    for (int i = 1; i < MAX_SHARED_X; ++i) {
        const bool on = shared && i < shared->n;
        p.A_more[i - 1] = on ? (const char *)shared->A_stack[i] : nullptr;
        p.uh_more[i - 1] = on ? (char *)shared->u_hi[i] : nullptr;
        p.ul_more[i - 1] = on ? (char *)shared->u_lo[i] : nullptr;
    }
    if (shared) {
        p.A_stack = (const char *)shared->A_stack[0];
        p.u_hi = (char *)shared->u_hi[0];
        p.u_lo = (char *)shared->u_lo[0];
    }
    p.n_tiles_n = p.tiles_per_proj * p.n_proj;
    const int64_t grid = (int64_t)pv.max_tiles * (TILE_M / bm) * p.n_tiles_n;
    return grid > 0x7ffffff0LL ? -1 : grid;
}

template <class C, bool QUANT = false>
static hipError_t launch_shrink_as(const PlanView &pv, const LinearArgs &a, hipStream_t stream, void *xq = nullptr,
                                   void *xs = nullptr, const SharedX *shared = nullptr)
{
    ShrinkKParams p;
    const int64_t grid = shrink_params(p, pv, a, shared, xq, xs, C::BM, C::BN);
    if (grid < 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL((shrink_kernel<C, QUANT>), dim3((unsigned)round_up8((int)grid)), dim3(C::NT),
                       C::SMEM_BYTES, stream, p);
    return hipGetLastError();
}

template <class C, int QW = 0>
static hipError_t launch_shrink_patch(const PlanView &pv, const LinearArgs &a, const SharedX *shared, hipStream_t stream,
                                      void *xq = nullptr, void *xs = nullptr)
{
    ShrinkKParams p;
    const int64_t grid = shrink_params(p, pv, a, shared, xq, xs, C::BM, C::BN);
    if (grid < 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL((shrink_patch_kernel<C, QW>), dim3((unsigned)round_up8((int)grid)), dim3(64 * (C::NW + QW)), C::SMEM_BYTES, stream, p);
    return hipGetLastError();
}

// Which form of shrink_patch_kernel: 16 (a wave by itself), 32, 64 (columns of the tiles below), or 0 where the larger tiles are
// as fast.  Us of the kernel, by 2048 / 5632, x in the Infinity Cache and adapters from HBM ("cold") or all of it at hand ("hot"):
//  * 16 up to two of its waves per compute unit.  Rank 64, against 32: 1890 tokens hot 8.6, 15.9 / 9.4, 18.3; 8192 tokens (1024 waves) cold 22.5,
//    56.6 / 17.7, 42.4.  At rank 16 and less up to the line of rank 32: 18 700 tokens cold 24.1, 61.5 / 24.6, 63.4 / larger tiles 27.5, 70.2.
//  * 32 (64 tokens x 32 columns) up to rank 64.  Rank 32, against the larger tiles, half of which is padding: 18 700 tokens (584 row
//    tiles) hot 18.5, 44 / 18.6, 50, cold 29.4, 75 / 30.2, 78; three projections cold 48.4 / 48.2.  Rank 64, 32 / 64 / larger: 8192 tokens (512 patches of
//    32 x 32) hot 10.9, 20.4 / 12.1, 22.4 / 16.0, 32.8, cold 17.7, 42.4 / 22.9, 50.1 / 22.0, 51.0.
//  * 64 (64 x 64).  Rank 64, two projections, 64 / larger: 8192 tokens by 5632 (1024 patches) hot 24.9 / 33.8, cold 53.6 / 53.1; 12 288
//    (1536) hot 40.9 / 39.7, cold 92 / 87.  Rank 128, whose larger tiles are four times as large: 8192 tokens hot 12.3, 24.3 / 28.7, 65.8,
//    cold 22.4, 53.6 / 46.7, 110; 12 288, two by 5632 (3072 patches) hot 81 / 90, cold 128 / 131; 18 700, two (4672) 141 / 129, 181 / 162.
//  * With codes, 16 / 32 (32 x 64) or 64 / larger: rank 64, 4700 tokens hot 15.2, 37 / 17.4, 37 / 32, 74, 8192 cold 29, 80 / 24, 57 / 39, 95,
//    12 288 (768 patches) cold 35, 91 (32) / 42, 108, 18 700 hot 30, 108 (32) / 34, 99; rank 128, 1890 tokens hot 10.2, 22 / 18.3, 38 / 39, 95,
//    8192 cold 41, 117 / 27, 70 / 50, 119, 12 288 (1536) 44, 115 (64) / 56, 135, 18 700 hot 37, 126 (64) / 45, 123.
static int shrink_patch(const PlanView &pv, const LinearArgs &a, int n_proj, bool codes)
{
    if (a.d_in % 64 || a.r > 128) return 0;
    const int64_t tiles = host_tiles(pv, 32), cus = compute_units();
    const int64_t patches = tiles * ((a.r + 31) / 32) * n_proj;
    if (tiles * ((a.r + 15) / 16) * n_proj <= 2 * cus) return 16;
    if (a.r > 64) return patches <= (codes ? 6 : 12) * cus ? 64 : 0;
    if (codes) return patches <= 3 * cus ? 32 : 0;
    if (a.r <= 32) return tiles > 3 * cus ? 0 : a.r <= 16 ? 16 : 32;
    return patches <= 2 * cus ? 32 : patches <= 4 * cus ? 64 : 0;
}

// The prefill shrink and the MXFP8 quantisation of x in one pass over x (r >= 1,
// d_in a multiple of 128).
hipError_t launch_prefill_shrink_quant(const PlanView &pv, const LinearArgs &a, void *xq, void *xs,
                                       hipStream_t stream)
{
    if (pv.max_tiles <= 0) return hipSuccess;
    if (a.r <= 0 || a.d_in % 128) return hipErrorInvalidValue;
    switch (shrink_patch(pv, a, 1, true)) {
    case 16: return launch_shrink_patch<CfgPatch16, 1>(pv, a, nullptr, stream, xq, xs);
    case 32: return launch_shrink_patch<CfgPatchWide, 4>(pv, a, nullptr, stream, xq, xs);
    case 64: return launch_shrink_patch<CfgPatch64, 4>(pv, a, nullptr, stream, xq, xs);
    }
    if (a.r > 64 && a.r <= 128) return launch_shrink_as<CfgShrinkDeep, true>(pv, a, stream, xq, xs);
    return launch_shrink_as<CfgShrinkDeep64, true>(pv, a, stream, xq, xs);
}

static hipError_t launch_prefill_shrink_any(const PlanView &pv, const LinearArgs &a, const SharedX *shared, hipStream_t stream)
{
    if (a.r <= 0 || pv.max_tiles <= 0) return hipSuccess;
    switch (shrink_patch(pv, a, shared ? shared->n : 1, false)) {
    case 16: return launch_shrink_patch<CfgPatch16>(pv, a, shared, stream);
    case 32: return launch_shrink_patch<CfgPatch32>(pv, a, shared, stream);
    case 64: return launch_shrink_patch<CfgPatch64>(pv, a, shared, stream);
    }
    if (a.d_in % 64 == 0 && a.r > 64 && a.r <= 128)
        return launch_shrink_as<CfgShrinkR128>(pv, a, stream, nullptr, nullptr, shared);
    if (a.d_in % 64 == 0) return launch_shrink_as<CfgShrinkDma>(pv, a, stream, nullptr, nullptr, shared);
    return launch_shrink_as<CfgShrink>(pv, a, stream, nullptr, nullptr, shared);
}

hipError_t launch_prefill_shrink(const PlanView &pv, const LinearArgs &a, hipStream_t stream)
{
    return launch_prefill_shrink_any(pv, a, nullptr, stream);
}

hipError_t launch_prefill_shrink_shared(const PlanView &pv, const LinearArgs &a, int n, const void *const *A_stack,
                                        void *const *u_hi, void *const *u_lo, hipStream_t stream)
{
    if (n < 1 || n > MAX_SHARED_X) return hipErrorInvalidValue;
    const SharedX sh{n, A_stack, u_hi, u_lo};
    return launch_prefill_shrink_any(pv, a, &sh, stream);
}

template <class C>
static hipError_t launch_linear_as(const LinearKParams &p0, int64_t m_tiles, hipStream_t stream)
{
    LinearKParams p = p0;
    p.n_tiles_n = (p.d_out + C::BN - 1) / C::BN;
    const int64_t total = m_tiles * p.n_tiles_n;
    if (total > 0x7ffffff0LL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(linear_kernel<C>, dim3((unsigned)round_up8((int)total)), dim3(C::NT),
                       C::SMEM_BYTES, stream, p);
    return hipGetLastError();
}

hipError_t launch_prefill_linear_shared(const PlanView &pv, const LinearArgs *a, int n, hipStream_t stream)
{
    if (pv.max_tiles <= 0) return hipSuccess;
    return launch_linear_stream_shared(pv, a, n, compute_units(), stream);
}

hipError_t launch_prefill_linear(const PlanView &pv, const LinearArgs &a, hipStream_t stream)
{
    if (pv.max_tiles <= 0) return hipSuccess;
    if (stream_kernel_fits(a)) return launch_linear_stream(pv, a, compute_units(), stream);
    if (mid_kernel_pays(pv, &a, 1, compute_units())) return launch_linear_mid(pv, &a, 1, compute_units(), stream);
    LinearKParams p;
    p.x = (const char *)a.x; p.W = (const char *)a.W; p.B_stack = (const char *)a.B_stack;
    p.u_hi = (const char *)a.u_hi; p.u_lo = (const char *)a.u_lo;
    p.y = (char *)a.y;
    p.tile_row0 = pv.tile_row0; p.tile_rows = pv.tile_rows; p.tile_expert = pv.tile_expert;
    p.tile_rank = pv.tile_rank;
    p.n_tiles = pv.n_tiles;
    p.T = pv.T;
    if (a.r > 0 && a.ldu != a.r) return hipErrorInvalidValue;   // (the tiled kernel's rows of u are r long)
    p.d_in = a.d_in; p.d_out = a.d_out; p.r = a.r;
    p.n_tiles_n = 0;
    p.y_f32 = a.y_f32;
    p.plain_tiles = 0;
    p.gather = nullptr;
    p.k_splits = 1; p.kb_per_split = 0;
    return launch_linear_as<CfgMain>(p, pv.max_tiles, stream);
}

// The decode base GEMM has few output tiles (T <= 1024 rows); cutting the
// contraction range gives the chip enough workgroups to keep many loads in
// flight.  The parts are summed, in order, by the expand kernel.
constexpr int DECODE_BASE_TARGET_WGS = 512;
constexpr int DECODE_BASE_MAX_SPLITS = 4;   // the expand kernel sums up to four parts
constexpr int DECODE_BASE_MIN_BLOCKS = 4;   // BK blocks per part at least
constexpr int DECODE_BASE_SPLIT_BLOCKS = 32;
// One row of tiles, not mixed with slabs (33 to 128 tokens): a block of a tile's loop takes 0.36 us however many loads are in
// flight (five stages instead of four change nothing), so up to four parts wherever they have this many blocks -- as long
// as the planes, which the expand reads back, are small.  By the projection's own width, not the call's: projections that
// share a call have the bits of calls of their own.  Us of a call, parts of 32 blocks / of 8 and more: 2048 -> 2048 rank 16 40
// tokens 19 / 15, 128 20 / 16, rank 128 64 of one sequence 20 / 15, 128 single 30 / 26; 1024 -> 1416 rank 64 64 21 / 15; 2048 -> 5632
// rank 16 40 22 / 19, 128 26 / 25, rank 128 128 43.5 / 42; 2048 -> 8192 rank 16 40 single 23 / 21, 80 27 / 26; beyond the line
// 128 of one sequence 23 / 25, 2048 -> 11008 rank 16 64 single 29 / 30, 2048 -> 22016 43 / 48.  What it costs: several wide projections in a call fill the chip
// with fewer parts, twice 2048 -> 5632 rank 16 40 26.0 / 27.2, rank 128 64 single 59 / 63, 64 of one sequence 25.2 / 25.0, twice 1024 -> 2816
// rank 64 128 single 30 / 33; in layers of 33 to 128 tokens, ranks 16 to 128, the others outweigh that (0.90 to 0.99 of the
// time; 64 to 128 single tokens at rank 128 1.01).
constexpr int DECODE_BASE_SPLIT_BLOCKS_FEW = 8, DECODE_BASE_FEW_MIN = 33, DECODE_BASE_FEW_MAX = 128;
constexpr int DECODE_BASE_FEW_OUT = 8192, DECODE_BASE_FEW_PLANE = DECODE_BASE_FEW_MAX * 5632;   // outputs; values of a plane
// Tokens up to which the rule for few takes this many outputs.
static int64_t few_tokens(int d_out)
{
    return d_out > DECODE_BASE_FEW_OUT ? 0 : std::min(DECODE_BASE_FEW_MAX, DECODE_BASE_FEW_PLANE / d_out);
}

template <class C>
static void shape_for(int64_t T, int d_in, int d_out, bool may_split, DecodeBaseShape *sh)
{
    sh->m_tiles = (T + C::BM - 1) / C::BM;
    sh->n_tiles_n = (d_out + C::BN - 1) / C::BN;
    const int64_t tiles = sh->m_tiles * sh->n_tiles_n;
    const int nkb = (d_in + C::BK - 1) / C::BK;
    int want = may_split ? (int)((DECODE_BASE_TARGET_WGS + tiles - 1) / (tiles > 0 ? tiles : 1)) : 1;
    if (want > DECODE_BASE_MAX_SPLITS) want = DECODE_BASE_MAX_SPLITS;
    // every part costs a plane of fp32 partial sums written and read back: no more
    // parts than it takes to keep a tile's serial loop to about DECODE_BASE_SPLIT_BLOCKS blocks
    const bool few = T >= DECODE_BASE_FEW_MIN && T <= few_tokens(d_out);
    const int blocks = few ? DECODE_BASE_SPLIT_BLOCKS_FEW : DECODE_BASE_SPLIT_BLOCKS;
    const int by_len = (nkb + blocks - 1) / blocks;
    if (want > by_len) want = by_len;
    if (want > nkb / DECODE_BASE_MIN_BLOCKS) want = nkb / DECODE_BASE_MIN_BLOCKS;
    if (want < 1) want = 1;
    const int per = (nkb + want - 1) / want;
    sh->kb_per_split = per;
    sh->k_splits = (nkb + per - 1) / per;   // no empty part
    sh->grid = round_up8((int)(tiles * sh->k_splits));
}

static DecodeBaseShape base_shape(int64_t T, int d_in, int d_out, bool may_split)
{
    DecodeBaseShape sh;
    sh.slab_blocks = 0;
    const int slabs = (d_out + 15) / 16;
    if (may_split && (T <= 16 || (T <= 32 && d_in <= BASE_SLAB_PIECE && slabs <= BASE_SLAB_MAX))) {
        sh.dma = 0;
        sh.slab_blocks = (int)((T + 15) / 16);
        sh.m_tiles = 1;
        sh.n_tiles_n = sh.grid = slabs;
        sh.k_splits = 1;
        sh.kb_per_split = (d_in + 31) / 32;
        return sh;
    }
    sh.dma = (d_in % 64 == 0);
    if (sh.dma) shape_for<CfgDecodeBase>(T, d_in, d_out, may_split, &sh);
    else shape_for<CfgThin>(T, d_in, d_out, may_split, &sh);
    return sh;
}

DecodeBaseShape decode_base_shape(int64_t T, int d_in, int d_out) { return base_shape(T, d_in, d_out, true); }

int decode_base_splits(int64_t T, int d_in, int d_out) { return decode_base_shape(T, d_in, d_out).k_splits; }

int64_t decode_base_rows(int64_t T, int d_in, int d_out)
{
    // The parts fall as the row tiles become more (shape_for), and where the rule for few tokens ends: the most rows are those
    // of T tokens, of the last batch of few, or of the last that leaves room for two, three or four parts.
    const bool dma = d_in % 64 == 0;
    const int64_t bm = dma ? CfgDecodeBase::BM : CfgThin::BM, bn = dma ? CfgDecodeBase::BN : CfgThin::BN, cols = (d_out + bn - 1) / bn;
    int64_t most = T * decode_base_splits(T, d_in, d_out);
    auto try_ = [&](int64_t t) {
        if (t > 0 && t < T) most = std::max(most, t * decode_base_splits(t, d_in, d_out));
    };
    try_(few_tokens(d_out));
    for (int parts = 2; parts <= DECODE_BASE_MAX_SPLITS; ++parts) try_((DECODE_BASE_TARGET_WGS - 1) / (parts - 1) / cols * bm);
    return most;
}

LinearKParams decode_base_params(const PlanView &pv, const LinearArgs &a, void *out, int out_f32,
                                 const DecodeBaseShape &sh, const int *gather)
{
    LinearKParams p;
    p.x = (const char *)a.x; p.W = (const char *)a.W; p.B_stack = nullptr;
    p.u_hi = nullptr; p.u_lo = nullptr;
    p.y = (char *)out;
    p.tile_row0 = nullptr; p.tile_rows = nullptr; p.tile_expert = nullptr; p.tile_rank = nullptr;
    p.n_tiles = nullptr;
    p.T = pv.T;
    p.d_in = a.d_in; p.d_out = a.d_out; p.r = 0;
    p.n_tiles_n = sh.n_tiles_n;
    p.y_f32 = out_f32;
    p.plain_tiles = 1;
    p.gather = gather;
    p.k_splits = sh.k_splits; p.kb_per_split = sh.kb_per_split;
    return p;
}

static hipError_t launch_plain(const PlanView &pv, const LinearArgs &a, void *out, int out_f32,
                               const DecodeBaseShape &sh, const int *gather, hipStream_t stream)
{
    if (pv.T <= 0) return hipSuccess;
    const LinearKParams p = decode_base_params(pv, a, out, out_f32, sh, gather);
    if (sh.dma)
        hipLaunchKernelGGL(linear_kernel<CfgDecodeBase>, dim3((unsigned)sh.grid), dim3(CfgDecodeBase::NT),
                           CfgDecodeBase::SMEM_BYTES, stream, p);
    else
        hipLaunchKernelGGL(linear_kernel<CfgThin>, dim3((unsigned)sh.grid), dim3(CfgThin::NT),
                           CfgThin::SMEM_BYTES, stream, p);
    return hipGetLastError();
}

hipError_t launch_decode_base(const PlanView &pv, const DecodeArgs &d, hipStream_t stream)
{
    const DecodeBaseShape sh = decode_base_shape(pv.T, d.lin.d_in, d.lin.d_out);
    if (sh.k_splits != d.k_splits || sh.slab_blocks) return hipErrorInvalidValue;
    return launch_plain(pv, d.lin, d.ybase, 1, sh, pv.tok_sorted, stream);   // partial sums in by-expert order
}

hipError_t launch_decode_base_only(const PlanView &pv, const LinearArgs &a, hipStream_t stream)
{
    return launch_plain(pv, a, a.y, a.y_f32, base_shape(pv.T, a.d_in, a.d_out, false), nullptr, stream);
}

}  // namespace moin
