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

// u for 8 consecutive columns, the first `left` of which exist (the others are zeros), as a bf16 pair.
__device__ __forceinline__ void u_pair(const f32x4_t (&v)[2], int left, int act, float s, uint4 &hi, uint4 &lo)
{
    uint32_t h[8], l[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float f = q < left ? adapter_act(v[q >> 2][q & 3], act) * s : 0.f;
        h[q] = f32_to_bf16_bits(f);
        l[q] = f32_to_bf16_bits(f - bf16_bits_to_f32(h[q]));
    }
    hi = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
    lo = make_uint4(l[0] | (l[1] << 16), l[2] | (l[3] << 16), l[4] | (l[5] << 16), l[6] | (l[7] << 16));
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
    // variant of this kernel, so that a row's sum depends neither on how the experts are numbered
    // nor on which variant ran.
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
        uint4 oh, ol;
        const f32x4_t v2[2] = {{v[0], v[1], v[2], v[3]}, {v[4], v[5], v[6], v[7]}};
        u_pair(v2, re - n0 - col, act, s, oh, ol);
        const int64_t off = (int64_t)row * ldu + (int64_t)(n0 + col) * 2;
        *reinterpret_cast<uint4 *>(uh + off) = oh;
        *reinterpret_cast<uint4 *>(ul + off) = ol;
    });
}

// The shrink of a batch with few row tiles.  Bound by the chain of a tile's blocks, which a 64 x 64 tile of the kernel
// above works off one by one, behind a barrier each, at 0.4 us (32 x 32 accumulators that wait for their own reads and
// for themselves), on as many compute units as there are tiles.  Here a tile is 32 tokens by the whole rank (BN columns),
// and its four waves take every fourth block each, through stages of their own, so that there is no barrier until
// their sums meet in LDS.  (The waves' blocks lie side by side: 512 bytes of a row at a time.)
// Us of the kernel, above / this: 1890 tokens by 2048 at rank 64 15.4 / 8.6, at rank 128 25 / 15, by 5632 at rank 64 31 / 14, at
// rank 128 64 / 27; with codes as well, 1890 by 2048 at rank 64 32 / 17, 8192 by 5632 80 / 41.
template <int BN_>
struct SplitCfg {
    static constexpr int NW = 4, NT = NW * 64, BM = 32, BN = BN_, BK = 64, ROWB = BK * 2;
    static constexpr int A_I = BM / 8, B_I = BN / 8, LPB = A_I + B_I;       // requests per block, 8 rows each
    static constexpr int A_BYTES = BM * ROWB, STAGE_BYTES = (BM + BN) * ROWB;
    static constexpr int WAVE_BYTES = 160 * 1024 / NW, NS = WAVE_BYTES / STAGE_BYTES;   // 5, 3 or 2 stages
    static constexpr int PITCH = BN + 4;                                    // of the waves' sums, in floats
    static constexpr int SMEM_BYTES = NW * WAVE_BYTES;
    static_assert(BM * PITCH * 4 <= WAVE_BYTES && (NS - 1) * LPB < 64, "");
};

// QUANT: as above, x in MXFP8 as well, from the blocks in LDS; also of tiles without an adapter.
template <int BN, bool QUANT>
__global__ __launch_bounds__(256) void shrink_split_kernel(ShrinkKParams p)
{
    using C = SplitCfg<BN>;
    extern __shared__ __align__(16) char smem[];
    constexpr int SUB = TILE_M / C::BM;
    const int ntm = uniform(*p.n_tiles) * SUB;
    const int id = xcd_band_id(blockIdx.x, ntm * p.n_tiles_n);
    if (id < 0) return;
    const int tm = uniform(id / p.n_tiles_n), proj = uniform(id % p.n_tiles_n);
    const int t = tm / SUB, sub = tm % SUB;
    const int e = uniform(p.tile_expert[t]);
    const int rows = min(uniform(p.tile_rows[t]) - sub * C::BM, C::BM);
    const int re = min(p.r, uniform(p.tile_rank[t]));
    const bool shrink = e >= 0 && re > 0;
    if (rows <= 0 || (!QUANT && !shrink)) return;
    const int row0 = uniform(p.tile_row0[t]) + sub * C::BM;
    const char *A_stack = p.A_stack;
    char *u_hi = p.u_hi, *u_lo = p.u_lo;
#pragma unroll
    for (int i = 1; i < MAX_SHARED_X; ++i)
        if (proj == i) {
            A_stack = p.A_more[i - 1];
            u_hi = p.uh_more[i - 1];
            u_lo = p.ul_more[i - 1];
        }
    const int r_out = min(p.ldu, (re + 63) & ~63);   // columns of u to write, zeros from the rank on
    const uint32_t ldx = (uint32_t)p.d_in * 2u;
    const char *xa = p.x + (int64_t)row0 * ldx;
    // (a walk for the quantiser alone puts x in A_e's place: valid addresses, unused products)
    const char *ae = shrink ? A_stack + (int64_t)e * p.r * ldx : xa;
    const int a_rows = shrink ? re : rows;
    const int nkb = p.d_in / C::BK;
    const int k_first = (int)(((uint32_t)(row0 - sub * C::BM) / (uint32_t)TILE_M * 5u) % (uint32_t)nkb);

    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    char *const mine = smem + wave * C::WAVE_BYTES;
    // as in DmaCore: 8 rows of 128 bytes a request, 16-byte chunks XORed with swz(row) = (row >> 1) & 7
    const uint32_t c16a = (((uint32_t)lane & 7) ^ ((uint32_t)lane >> 4)) * 16, c16b = c16a ^ 64u;   // even, odd requests
    uint32_t off[C::LPB];
#pragma unroll
    for (int j = 0; j < C::LPB; ++j) {
        const bool a = j < C::A_I;
        const int row = (a ? j : j - C::A_I) * 8 + (lane >> 3);
        off[j] = (uint32_t)min(row, (a ? rows : a_rows) - 1) * ldx + ((j & 1) ? c16b : c16a);
    }
    const int nb = (nkb - wave + C::NW - 1) / C::NW;   // the wave's blocks
    auto block_of = [&](int i) __attribute__((always_inline)) {
        const int kb = k_first + wave + i * C::NW;
        return kb >= nkb ? kb - nkb : kb;
    };
    auto issue = [&](int i) __attribute__((always_inline)) {
        const int kb = block_of(i);
        char *st = mine + (i % C::NS) * C::STAGE_BYTES;
#pragma unroll
        for (int j = 0; j < C::LPB; ++j)
            __builtin_amdgcn_global_load_lds(MOIN_GPTR((j < C::A_I ? xa : ae) + (off[j] + (uint32_t)kb * C::ROWB)),
                                             MOIN_LPTR(st + j * 1024), 16, 0, 0);
    };
    constexpr int FN = BN / 32;
    f32x16_t acc[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;
    const int r32 = lane & 31, h = lane >> 5, f = (r32 >> 1) & 7;
#pragma unroll
    for (int s = 0; s < C::NS; ++s)
        if (s < nb) issue(s);
    for (int i = 0; i < nb; ++i) {
        if (i + C::NS <= nb) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((C::NS - 1) * C::LPB) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const char *st = mine + (i % C::NS) * C::STAGE_BYTES;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int o = ((ks * 2 + h) ^ f) * 16;
            const bf16x8_t a = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(st + r32 * C::ROWB + o));
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const bf16x8_t b = __builtin_bit_cast(
                    bf16x8_t, *reinterpret_cast<const uint4 *>(st + C::A_BYTES + (j * 32 + r32) * C::ROWB + o));
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[j], 0, 0, 0);
            }
        }
        if constexpr (QUANT) {
            const int k0 = block_of(i) * C::BK, c = lane & 7;
#pragma unroll
            for (int j = 0; j < C::A_I; ++j) {
                const int row = j * 8 + (lane >> 3);
                int E;
                const uint2 codes = mx_quantize8(
                    *reinterpret_cast<const uint4 *>(st + row * C::ROWB + ((c ^ ((row >> 1) & 7)) * 16)), E);
                const uint32_t pair = (uint32_t)E | ((uint32_t)dpp_move<DPP_FROM_PLUS4>(E) << 8);
                if (row < rows) {
                    *reinterpret_cast<uint2 *>(p.xq + (int64_t)(row0 + row) * p.d_in + k0 + c * 8) = codes;
                    if (c == 0)
                        *reinterpret_cast<uint16_t *>(p.xs + ((int64_t)(k0 >> 7) * p.T + row0 + row) * 4 + ((k0 >> 5) & 3)) =
                            (uint16_t)pair;
                }
            }
        }
        // (the stage's reads have returned: the products above took them)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (i + C::NS < nb) issue(i + C::NS);
    }
    if (!shrink) return;   // (the whole workgroup)
    float *sum = reinterpret_cast<float *>(mine);
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) sum[mfma32_acc_row(q, lane) * C::PITCH + j * 32 + r32] = acc[j][q];
    __syncthreads();
    const int64_t ldu = (int64_t)p.ldu * 2;
    constexpr int COLS = BN < 64 ? 64 : BN;   // (u goes to the end of a block of 64)
    for (int i = threadIdx.x; i < C::BM * (COLS / 8); i += C::NT) {
        const int row = i / (COLS / 8), col = i % (COLS / 8) * 8;
        if (row >= rows || col >= r_out) continue;
        f32x4_t v[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        if (col < BN)
#pragma unroll
            for (int w = 0; w < C::NW; ++w)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    v[q] += *reinterpret_cast<const f32x4_t *>(smem + w * C::WAVE_BYTES + (row * C::PITCH + col + q * 4) * 4);
        uint4 hi, lo;
        u_pair(v, re - col, p.act, p.scale, hi, lo);
        const int64_t at = (int64_t)(row0 + row) * ldu + (int64_t)col * 2;
        *reinterpret_cast<uint4 *>(u_hi + at) = hi;
        *reinterpret_cast<uint4 *>(u_lo + at) = lo;
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
    if ((e = allow_lds(&shrink_split_kernel<64, true>, SplitCfg<64>::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_split_kernel<128, true>, SplitCfg<128>::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_split_kernel<32, false>, SplitCfg<32>::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_split_kernel<64, false>, SplitCfg<64>::SMEM_BYTES)) != hipSuccess) return e;
    if ((e = allow_lds(&shrink_split_kernel<128, false>, SplitCfg<128>::SMEM_BYTES)) != hipSuccess) return e;
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

template <int BN, bool QUANT = false>
static hipError_t launch_shrink_split(const PlanView &pv, const LinearArgs &a, const SharedX *shared, hipStream_t stream,
                                      void *xq = nullptr, void *xs = nullptr)
{
    using C = SplitCfg<BN>;
    ShrinkKParams p;
    const int64_t grid = shrink_params(p, pv, a, shared, xq, xs, C::BM, BN);
    if (grid < 0 || p.tiles_per_proj != 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL((shrink_split_kernel<BN, QUANT>), dim3((unsigned)round_up8((int)grid)), dim3(C::NT), C::SMEM_BYTES, stream, p);
    return hipGetLastError();
}

// Whether the whole rank in tiles of 32 tokens, `tiles` of them at most (of sequences of equal length, as far as the host
// knows), is the faster form.  The order in which u is summed differs between the forms, so the rule looks at the batch alone and not at
// how many projections the call has: a shared call gives the bits of the single ones, and on a quantised base codes
// made on the way give those of codes that were there.
static bool shrink_split_pays(const PlanView &pv, const LinearArgs &a, int tiles)
{
    if (a.d_in % 64 || a.r > 128) return false;
    const int64_t S = std::max<int64_t>(1, std::min<int64_t>(pv.S, pv.max_tiles)), len = (pv.T + S - 1) / S;
    return S * ((len + 31) / 32) <= tiles;
}

// The prefill shrink and the MXFP8 quantisation of x in one pass over x (r >= 1,
// d_in a multiple of 128).
hipError_t launch_prefill_shrink_quant(const PlanView &pv, const LinearArgs &a, void *xq, void *xs,
                                       hipStream_t stream)
{
    if (pv.max_tiles <= 0) return hipSuccess;
    if (a.r <= 0 || a.d_in % 128) return hipErrorInvalidValue;
    if (shrink_split_pays(pv, a, compute_units()))
        return a.r <= 64 ? launch_shrink_split<64, true>(pv, a, nullptr, stream, xq, xs)
                         : launch_shrink_split<128, true>(pv, a, nullptr, stream, xq, xs);
    if (a.r > 64 && a.r <= 128) return launch_shrink_as<CfgShrinkDeep, true>(pv, a, stream, xq, xs);
    return launch_shrink_as<CfgShrinkDeep64, true>(pv, a, stream, xq, xs);
}

static hipError_t launch_prefill_shrink_any(const PlanView &pv, const LinearArgs &a, const SharedX *shared, int split_tiles,
                                            hipStream_t stream)
{
    if (a.r <= 0 || pv.max_tiles <= 0) return hipSuccess;
    if (shrink_split_pays(pv, a, split_tiles)) {
        if (a.r <= 32) return launch_shrink_split<32>(pv, a, shared, stream);
        if (a.r <= 64) return launch_shrink_split<64>(pv, a, shared, stream);
        return launch_shrink_split<128>(pv, a, shared, stream);
    }
    if (a.d_in % 64 == 0 && a.r > 64 && a.r <= 128)
        return launch_shrink_as<CfgShrinkR128>(pv, a, stream, nullptr, nullptr, shared);
    if (a.d_in % 64 == 0) return launch_shrink_as<CfgShrinkDma>(pv, a, stream, nullptr, nullptr, shared);
    return launch_shrink_as<CfgShrink>(pv, a, stream, nullptr, nullptr, shared);
}

// The split form where a call of any number of projections gains or loses nothing by it.  Us, tiles above / split, rank 64
// and 128, by 2048: 4096 tokens, one projection 15.4 / 9.1 and 23 / 15, three 16 / 16.5 and 28 / 26; 5120 tokens, three
// 16.5 / 17 and 29 / 27.5; 6144, three 18 / 23 and 29 / 37.  Long rows, whose chains of blocks cost the tiles above the more,
// a tile per compute unit (a call, by 5632, 8192 tokens: one projection 67 / 54 and 99 / 65, two 69 / 67 and 100 / 86; three, which
// models have on their shorter rows, 73 / 81 and 101 / 107).
constexpr int SPLIT_LONG_ROWS = 4096;
static int split_tiles_of(int d_in)
{
    return d_in >= SPLIT_LONG_ROWS ? compute_units() : compute_units() * 5 / 8;
}

hipError_t launch_prefill_shrink(const PlanView &pv, const LinearArgs &a, hipStream_t stream)
{
    return launch_prefill_shrink_any(pv, a, nullptr, split_tiles_of(a.d_in), stream);
}

hipError_t launch_prefill_shrink_shared(const PlanView &pv, const LinearArgs &a, int n, const void *const *A_stack,
                                        void *const *u_hi, void *const *u_lo, hipStream_t stream)
{
    if (n < 1 || n > MAX_SHARED_X) return hipErrorInvalidValue;
    const SharedX sh{n, A_stack, u_hi, u_lo};
    return launch_prefill_shrink_any(pv, a, &sh, split_tiles_of(a.d_in), stream);
}

// On a quantised base every call is of one projection: a tile per compute unit.  (Us of a call, tiles above / split, 8192
// tokens by 2048 at rank 64 42 / 37, with codes 58 / 45; 12 288 tokens 43 / 44 and 59 / 57.)
hipError_t launch_prefill_shrink_mx(const PlanView &pv, const LinearArgs &a, hipStream_t stream)
{
    return launch_prefill_shrink_any(pv, a, nullptr, compute_units(), stream);
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
    const int by_len = (nkb + DECODE_BASE_SPLIT_BLOCKS - 1) / DECODE_BASE_SPLIT_BLOCKS;
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
