// Decode path of the routed LoRA linear layer: a handful of tokens per
// sequence, hundreds of distinct adapters per batch, so the time goes into
// streaming W_a and W_b of every distinct adapter from HBM once (Section 1:
// many small adapters served together; Section 3.2: y = W x + W_b (W_a x)).
//
// Tokens arrive grouped by expert (plan), in records of at most `chunk` tokens.  An item of work is a slab of one
// record's adapter rows against its (at most a few) tokens with v_mfma_f32_16x16x32_bf16, whose 16 columns are 16
// tokens.  Idle MFMA columns cost nothing here: the kernels are HBM-bound, and what decides their speed is
//  * how the adapter is asked for: 512 consecutive bytes of a row or more per instruction, non-temporal, and into the
//    MFMA operand's order through LDS of the wave's own.  The operand's map as a load (16 rows x 64 bytes per
//    instruction) reads 400 adapters of 512 KB at 5.6 TB/s, 3.5 when the Infinity Cache is full of dirty lines (as
//    after a base product); this one at 6.3 and 6.1, it leaves that cache alone (operand map and non-temporal: 5.4).
//  * that loads are always in flight: a workgroup (a wave, in the expand) walks through items, the next one's
//    adapter rows going out before the present one's are waited for (two sets of registers, in turn; a step after the
//    last, or without an adapter, loads a few bytes that nobody uses, so that the number of loads in flight is the same
//    on every path and the compiler can wait for the older ones alone);
//  * that no workgroup is launched for nothing: the number of distinct experts is known on the device only (a batch
//    of 1024 Zipf-drawn sequences has 340), and a workgroup for a record that is not there costs a slot and a trip to
//    memory.  The grids are sized for the chip.
// Records of several token blocks (longer sequences) keep their slab in registers instead (the "held" kernels).
//
//   base   : ybase[s] = x[:, range s] W[:, range s]^T   (fp32; tiles of linear_tile.h, or slabs in the smallest batches)
//   shrink : ug[pos, :] = scale * A_e x_tok             (bf16 high part + remainder)
//   expand : y[tok, :]  = sum_s ybase[s][tok, :] + B_e ug[pos]
#include <algorithm>

#include "gemm_core.h"
#include "kernels.h"
#include "linear_tile.h"

namespace moin {

// 16-byte operand fragment at row + k*2 bytes.  Past the row end (k >= klen)
// the load is redirected to k = 0 and the data zeroed, so no branch is needed.
// Lanes whose row is only padding pass any in-bounds row: an MFMA output
// depends on its own row and column only, and padded outputs are not stored.
__device__ __forceinline__ bf16x8_t ldg_frag(const char *row, int k, int klen)
{
    const bool ok = k < klen;
    const uint32_t m = ok ? 0xFFFFFFFFu : 0u;
    uint4 v = *reinterpret_cast<const uint4 *>(row + (ok ? k : 0) * 2);
    v.x &= m; v.y &= m; v.z &= m; v.w &= m;
    return __builtin_bit_cast(bf16x8_t, v);
}

// Group records and the token indices of a block come through the scalar cache: a
// scalar load does not queue behind the compute unit's vector-memory traffic, so a
// workgroup knows its adapter and its tokens a few hundred nanoseconds after it starts
// and can then issue ALL of its vector loads at once -- one trip to memory per item
// instead of a chain of three.  (Under load every dependent vector load costs a full
// queueing delay of several microseconds.)  Reading through the constant address space
// at a uniform address is what makes a load a scalar one.
typedef int i32x2_t __attribute__((ext_vector_type(2)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x16_t __attribute__((ext_vector_type(16), aligned(4)));
#define MOIN_CONST_AS __attribute__((address_space(4)))
__device__ __forceinline__ int sload_x1(const int *p) { return *(const MOIN_CONST_AS int *)(uintptr_t)p; }
__device__ __forceinline__ i32x2_t sload_x2(const int *p) { return *(const MOIN_CONST_AS i32x2_t *)(uintptr_t)p; }
__device__ __forceinline__ i32x4_t sload_x4(const int4 *p) { return *(const MOIN_CONST_AS i32x4_t *)(uintptr_t)p; }
__device__ __forceinline__ i32x16_t sload_x16(const int *p) { return *(const MOIN_CONST_AS i32x16_t *)(uintptr_t)p; }
// Element (lane % 16) of sixteen wave-uniform values.
__device__ __forceinline__ int pick16(const i32x16_t &t, int lane)
{
    const int i = lane & 15;
    int v = t[0];
#pragma unroll
    for (int k = 1; k < 16; ++k) v = (i == k) ? t[k] : v;
    return v;
}

// ldg_frag in two halves, so that a kernel can first issue every load it will need
// and only then touch the data (a scheduling barrier between the two keeps the
// compiler from waiting on one load before it has issued the next).
__device__ __forceinline__ uint4 ldg_raw(const char *row, int k, int klen)
{
    return *reinterpret_cast<const uint4 *>(row + (k < klen ? k : 0) * 2);
}
__device__ __forceinline__ bf16x8_t frag_of(uint4 v, int k, int klen)
{
    const uint32_t m = k < klen ? 0xFFFFFFFFu : 0u;
    v.x &= m; v.y &= m; v.z &= m; v.w &= m;
    return __builtin_bit_cast(bf16x8_t, v);
}

constexpr int SHRINK_WAVES = 8;   // waves of a workgroup split the d_in range
constexpr int SHRINK_BATCH = 8;   // k-steps (of 32) whose loads are issued together

struct ShrinkDParams {
    const char *x, *A_stack;
    char *ug_hi, *ug_lo;
    const int *tok_sorted;
    const int4 *grp_meta;
    const int *n_groups;
    int d_in, r;
    float scale;
    int act;
};

typedef float Partials[SHRINK_WAVES][64][4] __attribute__((aligned(16)));   // of one 16 x 16 block, a wave's share each

// Added in wave order: runs repeat bit for bit.
__device__ __forceinline__ f32x4_t sum_partials(const Partials &red, int lane)
{
    f32x4_t f = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < SHRINK_WAVES; ++w) f += *reinterpret_cast<const f32x4_t *>(red[w][lane]);
    return f;
}

// u for one block of 16 positions and 16 rows of A_e from the waves' partial sums, as a bf16 pair.  One wave calls it.
__device__ __forceinline__ void store_u(const Partials &red, int lane, int pos0, int ge, int j0, int r, int ldr, int act,
                                        float scale, char *ug_hi, char *ug_lo)
{
    // lane holds u[token = lane % 16][j0 + 4 * (lane / 16) + i]
    const f32x4_t s = sum_partials(red, lane);
    uint32_t h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float f = adapter_act(s[i], act) * scale;
        h[i] = f32_to_bf16_bits(f);
        l[i] = f32_to_bf16_bits(f - bf16_bits_to_f32(h[i]));
    }
    const int pos = pos0 + (lane & 15), jj = j0 + 4 * (lane >> 4);
    if (pos < ge && jj < r) {   // r % 8 == 0, so a group of 4 is all in or all out
        const int64_t off = ((int64_t)pos * ldr + jj) * 2;
        *reinterpret_cast<uint2 *>(ug_hi + off) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
        *reinterpret_cast<uint2 *>(ug_lo + off) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
    }
}

// One (expert group g, 16-row slab of A_e) of a large batch's shrink; `red` is two buffers, used in turn (`flip`).
// KS_HOLD > 0 (records of several blocks of 16 tokens): a wave's share of the slab is at
// most KS_HOLD k-steps and stays in registers for all of the record's token
// blocks, instead of being fetched again for each.
template <int UNR, int KS_HOLD>
__device__ __forceinline__ void decode_shrink_slab(const ShrinkDParams &p, int slab, int g, Partials *red, int &flip)
{
    static_assert(KS_HOLD > 0 && KS_HOLD % UNR == 0, "whole batches");
    constexpr int NW = SHRINK_WAVES;
    const char *__restrict__ x = p.x;
    const char *__restrict__ A_stack = p.A_stack;
    const int *__restrict__ tok_sorted = p.tok_sorted;
    const int d_in = p.d_in;
    const i32x4_t gm = sload_x4(p.grp_meta + g);
    const int e = gm.x, gs = gm.y, ge = gm.z;
    // the expert's own rank (a multiple of 8): slabs beyond it are never read, u is
    // stored [pos, p.r] and only its first r columns are written and later read
    const int r = min(p.r, gm.w);
    if (e < 0 || ge <= gs || slab * 16 >= r) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j0 = slab * 16;
    const int jrow = j0 + (lane & 15);
    const int kq = (lane >> 4) * 8;               // element offset of this lane's k-group
    const int64_t ld = (int64_t)d_in * 2;
    const char *arow = A_stack + ((int64_t)e * p.r + (jrow < r ? jrow : 0)) * ld;
    // each wave owns a contiguous run of k-steps: its 16 rows are read as 16
    // contiguous segments
    const int nks = (d_in + 31) / 32;
    const int per = (nks + NW - 1) / NW;
    const int ks_beg = wave * per;
    const int ks_end = min(nks, ks_beg + per);
    const int klen = min(d_in, ks_end * 32);

    bf16x8_t held[KS_HOLD];
#pragma unroll
    for (int u = 0; u < KS_HOLD; ++u) held[u] = ldg_frag(arow, (ks_beg + u) * 32 + kq, klen);   // past the range: zero
    for (int t0 = gs; t0 < ge; t0 += 16) {
        // (entries past the record's end are read -- the list is followed by more of the plan -- and not used: such
        // lanes take the block's first token, in bounds, result unused)
        const i32x16_t toks = sload_x16(tok_sorted + t0);
        const int tok = t0 + (lane & 15) < ge ? pick16(toks, lane) : toks[0];
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
        const char *xrow = x + (int64_t)tok * ld;
#pragma unroll
        for (int u0 = 0; u0 < KS_HOLD; u0 += UNR) {
            if (ks_beg + u0 < ks_end) {   // the same for the whole wave
                bf16x8_t b[UNR];
#pragma unroll
                for (int u = 0; u < UNR; ++u) b[u] = ldg_frag(xrow, (ks_beg + u0 + u) * 32 + kq, klen);
#pragma unroll
                for (int u = 0; u < UNR; ++u)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(held[u0 + u], b[u], acc, 0, 0, 0);
            }
        }
        Partials &part = red[flip & 1];
#pragma unroll
        for (int i = 0; i < 4; ++i) part[wave][lane][i] = acc[i];
        lds_barrier();   // (one is enough: a buffer is written again only after the next one)
        if (wave == (flip & (NW - 1))) store_u(part, lane, t0, ge, j0, r, p.r, p.act, p.scale, p.ug_hi, p.ug_lo);
        ++flip;
    }
}

// What differs between the projections of one call that read the same x (gate, up; q, k, v): they
// share the token groups, d_in, r and the scale, so their base tiles, their shrink slabs and their expand
// blocks stand side by side in the call's two launches and the launches' ramp and tail are paid once.  Entry 0 repeats what the plain parameter blocks hold.
struct DecodeMore {
    int n;                          // projections of the call (1..MAX_SHARED_X)
    int tile_first[MAX_SHARED_X];   // first base tile of each (multiples of 8; the next one's where it has none)
    int slab_first[MAX_SHARED_X];   // first slab of W of each (likewise)
    int xb_first[MAX_SHARED_X];     // first expand row block of each
    int k_splits[MAX_SHARED_X];     // parts of each one's base product
    const char *W[MAX_SHARED_X], *A_stack[MAX_SHARED_X], *B_stack[MAX_SHARED_X];
    char *ug_hi[MAX_SHARED_X], *ug_lo[MAX_SHARED_X], *y[MAX_SHARED_X];
    float *ybase[MAX_SHARED_X];
    int d_out[MAX_SHARED_X], n_tiles_n[MAX_SHARED_X];
};

// Which items a workgroup of a persistent launch takes.  `n_base` long items (base products) go first, workgroup w
// taking numbers w, w + P, ...; each of them stands for `c` short ones (shrink slabs), which fill the turns that are
// left, also in the order of the workgroups: static, so that nothing has to be counted in memory, and even.
struct Turns {
    int P, n_base, c;
    __device__ __forceinline__ int short_item(int w, int j) const
    {
        const int rem = n_base % P;   // workgroups with one long item more than the others
        if (w < rem) return c * (P - rem) + j * P + w;
        if (j < c) return j * (P - rem) + (w - rem);
        return c * (P - rem) + (j - c) * P + w;
    }
};

constexpr int STREAM_KSTEPS = 8;                          // k-steps (of 32) per wave and step
constexpr int STREAM_COL = STREAM_KSTEPS * 64;            // bytes of a row that a wave takes in a step
constexpr int STREAM_STAGE = SHRINK_WAVES * 16 * STREAM_COL;   // 16 rows x 4 KB
constexpr int STREAM_SMEM = STREAM_STAGE + 2 * (int)sizeof(Partials);   // 80 KB: two workgroups per compute unit

// The same value, which the compiler cannot know: what is derived from it is computed where it is used and does not
// stay in registers across a streaming loop, whose loads in flight need them.
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// 16 bytes of an adapter, read once per call: not to displace what is in the Infinity Cache.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ldg_nt(const char *p)
{
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p)));
}

// The arguments of the streaming kernels, read back where they are needed from the kernel's argument block: uniform
// loads through the scalar cache, so that what a projection picks can be indexed and does not stay in registers.
struct ShrinkStreamArgs {
    ShrinkDParams sp;
    LinearKParams lp;
    DecodeMore m;
    Turns turns;
    int n_w, n_slabs, max_groups;
};
template <class A>
__device__ __forceinline__ const MOIN_CONST_AS A *kernel_args()
{
    const MOIN_CONST_AS int *words = (const MOIN_CONST_AS int *)__builtin_amdgcn_kernarg_segment_ptr();
    // A word of each of its 64-byte lines, together: one trip to memory, and later reads of the block find their line in
    // the scalar cache.
    constexpr int LINES = (sizeof(A) + 63) / 64;
    int v[LINES];
#pragma unroll
    for (int i = 0; i < LINES; ++i) v[i] = words[i * 16];
#pragma unroll
    for (int i = 0; i < LINES; ++i) asm volatile("" ::"s"(v[i]));
    return (const MOIN_CONST_AS A *)words;
}

// Number of records, how many of them are base-only, and the first record that a workgroup (a wave, in the expand) will
// want if none of them is: one trip to memory for both.
struct FirstRecord {
    i32x2_t recs;
    i32x4_t meta;
};
__device__ __forceinline__ FirstRecord first_record(const int *n_groups, const int4 *grp_meta, int g)
{
    FirstRecord f{sload_x2(n_groups), sload_x4(grp_meta + g)};
    asm volatile("" : "+s"(f.recs), "+s"(f.meta));
    return f;
}

// The shrink as one stream of loads per workgroup, two workgroups per compute unit.  An item is 16 rows of A_e of one
// (record, projection) -- or, in the smallest batches (decode_base_shape), 16 rows of W (`n_w` of them, first) against the whole
// batch: the base product is the same kind of work there.  A step is 4 KB of each of the 16 rows and one block of 16
// tokens: each wave owns 512 bytes of the rows and reads them as such, two rows per instruction; they take the MFMA
// operand's order in LDS of the wave's own, so there is no barrier but one per item, on LDS alone, where the waves'
// sums meet; one wave at a time adds them up.  The records' own loads (scalar) are an item ahead.
__device__ __forceinline__ void shrink_stream(const MOIN_CONST_AS ShrinkStreamArgs *args, char *smem)
{
    constexpr int NW = SHRINK_WAVES, KS = STREAM_KSTEPS;
    Partials *red = reinterpret_cast<Partials *>(smem + STREAM_STAGE);
    const int lane_id = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6), w = (int)blockIdx.x;
    char *const mine = smem + wave * (16 * STREAM_COL);
    const Turns turns{args->turns.P, args->turns.n_base, args->turns.c};
    const int n_w = args->n_w, n_slabs = args->n_slabs, r_stack = args->sp.r, d_in = args->sp.d_in;
    const int per_g = n_slabs * args->m.n;
    const int4 *grp_meta = args->sp.grp_meta;
    const int *tok_sorted = args->sp.tok_sorted;
    const char *x = args->sp.x;
    int turn = 0;
    int it_next = turns.short_item(w, 0);
    const FirstRecord fr =
        first_record(args->sp.n_groups, grp_meta, min(max(it_next - n_w, 0) / per_g, args->max_groups - 1));
    const int g_first = fr.recs.y;   // base-only records come first: nothing to do for them
    const int n_items = n_w + (fr.recs.x - g_first) * per_g;
    const uint32_t ld = (uint32_t)d_in * 2u;
    const int n_batches = (int)((ld + NW * STREAM_COL - 1) / (NW * STREAM_COL));
    const uint32_t col = (uint32_t)wave * STREAM_COL;

    struct Item {
        const char *A;           // first of the 16 rows
        int rows, t0, ge;        // rows that exist (0: nothing to do), the block's first position, one past the last
        int proj, j0, r;         // proj < 0: rows of W of projection ~proj; r: rank, or d_out
        int batch;               // the step's piece of the rows
        int kept;                // the rows are in LDS already: only the tokens change
    };
    if (it_next >= n_items) return;
    auto meta_of = [&](int it) __attribute__((always_inline)) {
        return sload_x4(grp_meta + (it >= n_w && it < n_items ? g_first + (it - n_w) / per_g : 0));
    };
    i32x4_t gm_next = g_first == 0 ? fr.meta : meta_of(it_next);
    bool more = true;
    // The workgroup's next item.  Past the expert's rank there is nothing to read, nor without an adapter.
    auto advance = [&]() __attribute__((always_inline)) {
        Item o;
        const int it = it_next;
        const i32x4_t gm = gm_next;
        more = it < n_items;
        it_next = turns.short_item(w, ++turn);
        gm_next = meta_of(it_next);
        o.batch = o.kept = 0;
        if (it < n_w) {
            int q = 0;
#pragma unroll
            for (int i = 1; i < MAX_SHARED_X; ++i) q += i < args->m.n && it >= args->m.slab_first[i];
            o.proj = ~q;
            o.j0 = (it - args->m.slab_first[q]) * 16;
            o.r = args->m.d_out[q];
            o.rows = min(16, o.r - o.j0);
            o.A = args->m.W[q] + (int64_t)o.j0 * ld;
            o.t0 = 0;
            o.ge = (int)args->lp.T;
        } else {
            const int idx = (it - n_w) % per_g;
            o.proj = idx / n_slabs;
            o.j0 = (idx - o.proj * n_slabs) * 16;
            o.t0 = gm.y;
            o.ge = gm.z;
            o.r = min(r_stack, gm.w);
            o.rows = more && gm.x >= 0 ? max(0, min(16, o.r - o.j0)) : 0;
            o.A = args->m.A_stack[o.proj] + ((int64_t)(o.rows > 0 ? gm.x : 0) * r_stack + (o.rows > 0 ? o.j0 : 0)) * ld;
        }
        return o;
    };
    // The wave's 16 x 512 bytes of a step's rows (instruction u: rows 2u and 2u + 1).  Past the rows or the row's end a
    // valid address is read instead and masked or never used.
    auto issue_rows = [&](const Item &o, uint4(&ra)[KS]) __attribute__((always_inline)) {
        const int lane = opaque(lane_id);
        const uint32_t ka = (uint32_t)o.batch * (NW * STREAM_COL) + col + (uint32_t)(lane & 31) * 16;
        const int rows = o.kept ? 0 : o.rows;
        const uint32_t kk = rows > 0 && ka < ld ? ka : 0u;
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            const int row = 2 * u + (lane >> 5);
            ra[u] = ldg_nt(o.A + ((row < rows ? (uint32_t)row * ld : 0u) + kk));
        }
    };
    auto toks_of = [&](const Item &o) __attribute__((always_inline)) {
        // (entries past the record's end are read -- the list is followed by more of the plan -- and not used)
        return sload_x16(tok_sorted + o.t0);
    };
    Item cur = advance();
    i32x16_t toks = toks_of(cur);
    int flip = 0;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    // One step: its rows are in flight to `ra`; the next one's go to `ra_next`.
    auto step = [&](uint4(&ra)[KS], uint4(&ra_next)[KS]) __attribute__((always_inline)) {
        const int lane = opaque(lane_id);
        const uint32_t k0 = (uint32_t)cur.batch * (NW * STREAM_COL) + col;
        // (lanes past the record's end take the block's first token)
        const int tok = cur.t0 + (lane & 15) < cur.ge ? pick16(toks, lane) : toks[0];
        const char *xrow = x + (int64_t)tok * ld;
        uint4 rx[KS];
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            const uint32_t k = k0 + (uint32_t)(u * 64 + (lane >> 4) * 16);
            rx[u] = *reinterpret_cast<const uint4 *>(xrow + (k < ld ? k : 0u));
        }
        const bool last = cur.batch + 1 == n_batches;
        Item nxt = cur;
        if (!last) ++nxt.batch;
        else if (cur.t0 + 16 < cur.ge) {   // several blocks
            nxt.t0 += 16;
            nxt.kept = n_batches == 1;
            nxt.batch = 0;
        }
        else nxt = advance();
        toks = toks_of(nxt);
        __builtin_amdgcn_sched_barrier(0);
        issue_rows(nxt, ra_next);
        __builtin_amdgcn_sched_barrier(0);
        const int ln = opaque(lane_id);
        // 16-byte chunk c of row j stands at place c ^ j: neither the writes (consecutive chunks) nor the operand's
        // reads (16 rows at one chunk) meet a bank twice
        if (!cur.kept) {
#pragma unroll
            for (int u = 0; u < KS; ++u) {
                const int row = 2 * u + (ln >> 5);
                *reinterpret_cast<uint4 *>(mine + row * STREAM_COL + (((ln & 31) ^ row) * 16)) = ra[u];
            }
        }
        const char *src = mine + (ln & 15) * STREAM_COL;
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            const uint4 fa = *reinterpret_cast<const uint4 *>(src + (((u * 4 + (ln >> 4)) ^ (ln & 15)) * 16));
            const int k = (int)(k0 >> 1) + u * 32 + (ln >> 4) * 8;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_of(fa, k, d_in), frag_of(rx[u], k, d_in), acc, 0, 0, 0);
        }
        if (last) {
            Partials &part = red[flip & 1];
            const int le = opaque(lane_id);
            *reinterpret_cast<f32x4_t *>(part[wave][le]) = acc;
            acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
            lds_barrier();   // (one is enough: a buffer is written again only after the next one)
            if (wave == (flip & (NW - 1)) && cur.rows > 0) {
                if (cur.proj < 0) {
                    const int pos = cur.t0 + (le & 15), o = cur.j0 + 4 * (le >> 4);
                    const f32x4_t v = sum_partials(part, le);
                    if (pos < cur.ge && o < cur.r)   // d_out % 8 == 0
                        *reinterpret_cast<f32x4_t *>(args->m.ybase[~cur.proj] + (int64_t)pos * cur.r + o) = v;
                } else {
                    store_u(part, le, cur.t0, cur.ge, cur.j0, cur.r, r_stack, args->sp.act, args->sp.scale,
                            args->m.ug_hi[cur.proj], args->m.ug_lo[cur.proj]);
                }
            }
            ++flip;
        }
        __builtin_amdgcn_sched_barrier(0);
        cur = nxt;
    };
    uint4 ra0[KS], ra1[KS];
    issue_rows(cur, ra0);
    for (;;) {
        step(ra0, ra1);
        if (!more) return;
        step(ra1, ra0);
        if (!more) return;
    }
}

// The shrink of a large batch: items of (record, 16 rows of A_e), the slabs of one expert neighbours in dispatch
// order, so its rows of A_e stream from HBM as one contiguous run.
template <int KS_HOLD>
__global__ __launch_bounds__(SHRINK_WAVES * 64) void decode_shrink_kernel(ShrinkDParams p, int n_slabs)
{
    __shared__ Partials red[2];
    const i32x2_t recs = sload_x2(p.n_groups);
    const int n_items = recs.x * n_slabs;
    int flip = 0;
    for (int it = recs.y * n_slabs + (int)blockIdx.x; it < n_items; it += (int)gridDim.x)
        decode_shrink_slab<SHRINK_BATCH, KS_HOLD>(p, it % n_slabs, it / n_slabs, red, flip);
}

// Base products and shrink slabs in one launch: the two are independent, the
// shrink is bound by HBM and the base tiles by latency, so side by side the base
// costs little time of its own.  TILES: base tiles of 128 x 128, each standing for
// turns.c items; else n_w slabs of 16 rows of W among the items (or none: the shrink alone).  With several projections
// in the call (`m`) the base work of all of them comes first.
static_assert(CfgDecodeBase::NT == SHRINK_WAVES * 64, "both roles share one workgroup size");
static_assert(CfgDecodeBase::SMEM_BYTES <= STREAM_SMEM, "the tiles' stages in the stream's LDS");
template <bool TILES, bool PACED>
__global__ __launch_bounds__(SHRINK_WAVES * 64, 4) void decode_base_shrink_kernel(ShrinkStreamArgs by_value)
{
    extern __shared__ __align__(16) char smem[];
    const MOIN_CONST_AS ShrinkStreamArgs *args = kernel_args<ShrinkStreamArgs>();
    if constexpr (TILES) {
        const int n_base = args->turns.n_base, P = args->turns.P;
        for (int b = (int)blockIdx.x; b < n_base; b += P) {
            int i = 0;
#pragma unroll
            for (int j = 1; j < MAX_SHARED_X; ++j) i += j < args->m.n && b >= args->m.tile_first[j];
            LinearKParams q = by_value.lp;
            q.W = args->m.W[i];
            q.y = reinterpret_cast<char *>(args->m.ybase[i]);
            q.d_out = args->m.d_out[i];
            q.n_tiles_n = args->m.n_tiles_n[i];
            q.k_splits = args->m.k_splits[i];
            q.kb_per_split = (q.d_in / CfgDecodeBase::BK + q.k_splits - 1) / q.k_splits;   // as decode_base_shape has it
            linear_tile<CfgDecodeBase, PACED>(q, b - args->m.tile_first[i], smem);
            __syncthreads();   // (the tile's epilogue has left LDS)
        }
    }
    shrink_stream(args, smem);
}

struct ExpandKParams {
    const char *B_stack, *ug_hi, *ug_lo;
    const float *ybase;        // [k_splits, T, d_out]
    char *y;
    const int *tok_sorted;
    const int4 *grp_meta;
    const int *n_groups;
    int64_t T;
    int d_out, r, k_splits, y_f32;
};

constexpr int EXPAND_WAVES = 4;

__device__ __forceinline__ void store_out(char *y, int d_out, int y_f32, int tok, int o, f32x4_t v)
{
    const int64_t at = (int64_t)tok * d_out + o;
    if (y_f32) {
        *reinterpret_cast<f32x4_t *>(y + at * 4) = v;
    } else {
        *reinterpret_cast<uint2 *>(y + at * 2) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
    }
}

// One (expert group, slab of EXPAND_WAVES * RB * 16 output rows).  KS_HOLD > 0:
// r <= 32 * KS_HOLD, the wave's RB x KS_HOLD fragments of B_e are requested at once
// and held across the group's token blocks; KS_HOLD == 0: any r, fragment by
// fragment.  The accumulators start from the base result, so y leaves in one pass.
// FULL (wave-uniform): the expert's rank is exactly 32 * KS_HOLD, so no fragment
// needs its tail cut off: loads take constant offsets from a few row addresses and
// nothing is masked.
// BY_POS: the rows of the base partial planes follow the by-expert token order (the
// small-batch base product gathers its rows that way), so nothing a workgroup
// loads depends on another load: adapter rows, u, base sums and token indices are
// all requested at once, and the token index is needed only to place the result.
// Phase 1 of a token block issues every load (for the first block also B_e, the HBM
// traffic); phase 2 consumes them; a scheduling barrier between the two keeps all
// loads ahead of the first wait.
template <int KS_HOLD, int NSPLIT, bool BY_POS, int RB, bool MIXED, bool FULL>
__device__ __forceinline__ void expand_item(const ExpandKParams &p, int slab, int e, int gs, int ge, int r)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int o_base = (slab * EXPAND_WAVES + wave) * (RB * 16);
    const int d_out = p.d_out;
    if (o_base >= d_out) return;
    const int kq = (lane >> 4) * 8;
    // rows of B_e and u are p.r long; the expert's own rank r (a multiple of 8) says how
    // much of them exists -- fragments past it are zero-filled, not read
    const int64_t ldb = (int64_t)p.r * 2;
    const char *bexp = p.B_stack + (int64_t)(e < 0 ? 0 : e) * d_out * ldb;
    const bool lora = e >= 0 && r > 0;
    constexpr int KH = KS_HOLD > 0 ? KS_HOLD : 1;
    auto ld_frag = [&](const char *row, int ks) __attribute__((always_inline)) -> uint4 {
        if constexpr (FULL) return *reinterpret_cast<const uint4 *>(row + ks * 64);   // row already at kq
        else return ldg_raw(row, ks * 32 + kq, r);
    };
    auto as_frag = [&](uint4 v, int ks) __attribute__((always_inline)) -> bf16x8_t {
        if constexpr (FULL) return __builtin_bit_cast(bf16x8_t, v);
        else return frag_of(v, ks * 32 + kq, r);
    };
    const int koff = FULL ? kq * 2 : 0;

    uint4 a[RB][KH];
    if constexpr (KS_HOLD > 0) {
        if (lora) {
#pragma unroll
            for (int c = 0; c < RB; ++c) {
                const int orow = o_base + c * 16 + (lane & 15);
                const char *brow = bexp + (int64_t)(orow < d_out ? orow : 0) * ldb + koff;
#pragma unroll
                for (int ks = 0; ks < KS_HOLD; ++ks) a[c][ks] = ld_frag(brow, ks);
            }
        }
    }

    for (int t0 = gs; t0 < ge; t0 += 16) {
        const int pos = t0 + (lane & 15);
        const bool tvalid = pos < ge;
        const int ps = tvalid ? pos : gs;
        const int tok = p.tok_sorted[ps];
        int brow_idx = ps;
        if constexpr (!BY_POS) brow_idx = tok;
        // lane holds y[token = lane % 16][o_base + c*16 + 4*(lane/16) + i]; rows
        // past d_out read (and never store) the last valid group of four
        f32x4_t part[RB][NSPLIT];
        {
            const int64_t plane = p.T * (int64_t)d_out;
#pragma unroll
            for (int c = 0; c < RB; ++c) {
                const int oo = min(o_base + c * 16 + 4 * (lane >> 4), d_out - 4);
                const float *src = p.ybase + (int64_t)brow_idx * d_out + oo;
#pragma unroll
                for (int sp = 0; sp < NSPLIT; ++sp)
                    part[c][sp] = *reinterpret_cast<const f32x4_t *>(src + (!MIXED || sp < p.k_splits ? sp * plane : 0));
            }
        }
        const char *uh = p.ug_hi + (int64_t)ps * ldb + koff;
        const char *ul = p.ug_lo + (int64_t)ps * ldb + koff;
        uint4 rh[KH], rl[KH];
        if constexpr (KS_HOLD > 0) {
            if (lora) {
#pragma unroll
                for (int ks = 0; ks < KS_HOLD; ++ks) {
                    rh[ks] = ld_frag(uh, ks);
                    rl[ks] = ld_frag(ul, ks);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);

        f32x4_t acc[RB];
#pragma unroll
        for (int c = 0; c < RB; ++c) {
            acc[c] = part[c][0];   // parts are added in order: repeatable
#pragma unroll
            for (int sp = 1; sp < NSPLIT; ++sp)
                if (!MIXED || sp < p.k_splits) acc[c] += part[c][sp];
        }
        if (lora) {
            if constexpr (KS_HOLD > 0) {
#pragma unroll
                for (int ks = 0; ks < KS_HOLD; ++ks) {
                    const bf16x8_t fh = as_frag(rh[ks], ks), fl = as_frag(rl[ks], ks);
#pragma unroll
                    for (int c = 0; c < RB; ++c) {
                        const bf16x8_t fa = as_frag(a[c][ks], ks);
                        acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fh, acc[c], 0, 0, 0);
                        acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fl, acc[c], 0, 0, 0);
                    }
                }
            } else {
                const int nks = (r + 31) / 32;
#pragma unroll
                for (int c = 0; c < RB; ++c) {
                    const int orow = o_base + c * 16 + (lane & 15);
                    const char *brow = bexp + (int64_t)(orow < d_out ? orow : 0) * ldb;
                    for (int ks = 0; ks < nks; ++ks) {
                        const int k = ks * 32 + kq;
                        const bf16x8_t ab = ldg_frag(brow, k, r);
                        const bf16x8_t bh = ldg_frag(p.ug_hi + (int64_t)ps * ldb, k, r);
                        const bf16x8_t bl = ldg_frag(p.ug_lo + (int64_t)ps * ldb, k, r);
                        acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ab, bh, acc[c], 0, 0, 0);
                        acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ab, bl, acc[c], 0, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int c = 0; c < RB; ++c) {
            const int oo = o_base + c * 16 + 4 * (lane >> 4);
            if (tvalid && oo < d_out) store_out(p.y, d_out, p.y_f32, tok, oo, acc[c]);   // d_out % 4 == 0
        }
    }
}

// Items of (record, EXPAND_WAVES * RB * 16 rows of B_e), the row blocks of one record neighbours; with several
// projections in the call (`m`) a record's items are the row blocks of all of them (n_xb).
// MIXED: projections with fewer parts of the base product than NSPLIT among them.
template <int KS_HOLD, int NSPLIT, bool BY_POS, int RB, bool MIXED>
__global__ __launch_bounds__(EXPAND_WAVES * 64) void decode_expand_kernel(ExpandKParams p, DecodeMore m, int n_xb)
{
    const int n_items = sload_x1(p.n_groups) * n_xb;
    for (int it = (int)blockIdx.x; it < n_items; it += (int)gridDim.x) {
        const int g = it / n_xb, xb = it - g * n_xb;
        const i32x4_t gm = sload_x4(p.grp_meta + g);
        const int e = gm.x, gs = gm.y, ge = gm.z;
        if (ge <= gs) continue;
        const int r = min(p.r, gm.w);
        ExpandKParams q = p;
        int first = 0;
#pragma unroll
        for (int i = 1; i < MAX_SHARED_X; ++i)
            if (i < m.n && xb >= m.xb_first[i]) {
                first = m.xb_first[i];
                q.B_stack = m.B_stack[i];
                q.ug_hi = m.ug_hi[i];
                q.ug_lo = m.ug_lo[i];
                q.ybase = m.ybase[i];
                q.y = m.y[i];
                q.d_out = m.d_out[i];
                q.k_splits = m.k_splits[i];
            }
        if (KS_HOLD > 0 && r == KS_HOLD * 32)
            expand_item<KS_HOLD, NSPLIT, BY_POS, RB, MIXED, true>(q, xb - first, e, gs, ge, r);
        else
            expand_item<KS_HOLD, NSPLIT, BY_POS, RB, MIXED, false>(q, xb - first, e, gs, ge, r);
    }
}

// The expand of batches whose records are mostly one block of 16 tokens: every wave walks through items of its own,
// 16 * RB rows of B_e of one (record, projection), one block of tokens at a time.  The rows are read as they lie (1 KB
// of consecutive bytes per instruction where r fills its k-steps) and take the operand's order in the wave's own LDS.
// KS: k-steps of 32 that the stacks' rank takes (1, 2 or 4).
// RB: at KS = 4 two, so that the small batches have items enough (8 single tokens, 2048 -> 5632 twice: 8.6 us, with four
// 10.3), but four beyond DECODE_MAX_T, where every item loads u and few tokens (8192 of them, 1558 experts: 547 us with
// two, 514); below, where the rows are short, always four.
constexpr int expand_stream_rb(int ks, bool large) { return ks <= 2 || large ? 4 : 2; }
// workgroups per compute unit, as the registers allow
constexpr int expand_stream_wgs(int ks, int parts, int rb)
{
    return ks == 1 ? (parts <= 2 ? 4 : 3) : ks == 2 ? (parts <= 2 ? 3 : 2) : rb > 2 ? 2 : parts == 1 ? 4 : 3;
}
constexpr int expand_stage(int ks, int rb) { return rb * 16 * ks * 64; }
struct ExpandStreamArgs {
    ExpandKParams p;
    DecodeMore m;
    int n_xb, max_groups;
};

// The base-only records (the first `n_rec`): y is the sum of the base product's parts.  Bound by memory; a wave takes 512
// consecutive columns of one token, whole lines per instruction.  (1024 base-only tokens through 2048 -> 5632, two parts:
// 10.5 us; as items like the others, 16 tokens by 32 rows of an adapter that is not there, 24.9.)
constexpr int BASE_ONLY_COLS = 512;
template <int NSPLIT, bool BY_POS, bool MIXED>
__device__ __forceinline__ void write_base_only(const MOIN_CONST_AS ExpandStreamArgs *args, int n_rec, int wave_id, int n_waves)
{
    constexpr int COLS = BASE_ONLY_COLS;
    struct Proj {
        const float *ybase;
        char *y;
        int d_out, splits;
    };
    const int lane = threadIdx.x & 63, y_f32 = args->p.y_f32, n = args->m.n;
    const int64_t T = args->p.T;
    const int *tok_sorted = args->p.tok_sorted;
    const int n_pos = sload_x4(args->p.grp_meta + n_rec - 1).z;
    const Proj only{args->p.ybase, args->p.y, args->p.d_out, NSPLIT};   // (most calls' one: its loads come all at once)
    auto blocks = [](int d_out) __attribute__((always_inline)) { return (d_out + COLS - 1) / COLS; };
    int per_pos = blocks(only.d_out);   // column blocks of all projections
    for (int i = 1; i < n; ++i) per_pos += blocks(args->m.d_out[i]);
    const uint32_t total = (uint32_t)n_pos * (uint32_t)per_pos;
    for (uint32_t u = wave_id; u < total; u += n_waves) {
        const int pos = (int)(u / (uint32_t)per_pos);
        const int tok = sload_x1(tok_sorted + pos);
        int c = (int)u - pos * per_pos;
        Proj q = only;
        if (n > 1) {
            int i = 0;
            for (; i + 1 < n && c >= blocks(args->m.d_out[i]); ++i) c -= blocks(args->m.d_out[i]);
            q = Proj{args->m.ybase[i], args->m.y[i], args->m.d_out[i], MIXED ? args->m.k_splits[i] : NSPLIT};
        }
        const float *src = q.ybase + (int64_t)(BY_POS ? pos : tok) * q.d_out;
        const int64_t plane = T * (int64_t)q.d_out;
        f32x4_t part[NSPLIT][2];
#pragma unroll
        for (int sp = 0; sp < NSPLIT; ++sp)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                part[sp][h] = *reinterpret_cast<const f32x4_t *>(src + (sp < q.splits ? sp * plane : 0) +
                                                                 min(c * COLS + h * (COLS / 2) + lane * 4, q.d_out - 4));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x4_t v = part[0][h];   // parts are added in order: repeatable
#pragma unroll
            for (int sp = 1; sp < NSPLIT; ++sp)
                if (sp < q.splits) v += part[sp][h];
            const int o = c * COLS + h * (COLS / 2) + lane * 4;
            if (o < q.d_out) store_out(q.y, q.d_out, y_f32, tok, o, v);   // d_out % 4 == 0
        }
    }
}

template <int KS, int NSPLIT, bool BY_POS, int RB, bool MIXED>
__device__ __forceinline__ void expand_stream(const MOIN_CONST_AS ExpandStreamArgs *args, char *smem, const FirstRecord &fr)
{
    constexpr int CPR = 4 * KS;   // 16-byte chunks per row
    const int lane_id = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6);
    char *const mine = smem + wave * expand_stage(KS, RB);
    const int n_xb = args->n_xb, r_stack = args->p.r, y_f32 = args->p.y_f32;
    const int4 *grp_meta = args->p.grp_meta;
    const int *tok_sorted = args->p.tok_sorted;
    const int g_first = fr.recs.y, n_items = (fr.recs.x - g_first) * n_xb;
    const int P = (int)gridDim.x * EXPAND_WAVES;
    const uint32_t ldb = (uint32_t)r_stack * 2u;
    const int64_t T = args->p.T;

    struct Item {
        const char *B;   // first of the rows
        int proj, o0, d_out, r, t0, ge;
        int kept;        // the rows are in LDS already: only the tokens change
    };
    int it_next = (int)blockIdx.x * EXPAND_WAVES + wave;
    if (it_next >= n_items) return;
    auto meta_of = [&](int it) __attribute__((always_inline)) { return sload_x4(grp_meta + (it < n_items ? g_first + it / n_xb : 0)); };
    i32x4_t gm_next = g_first == 0 ? fr.meta : meta_of(it_next);
    bool more = true;
    auto advance = [&]() __attribute__((always_inline)) {
        Item o;
        const int it = it_next;
        const i32x4_t gm = gm_next;
        more = it < n_items;
        it_next = it + P;
        gm_next = meta_of(it_next);
        const int xb = more ? it % n_xb : 0;
        o.proj = 0;
#pragma unroll
        for (int i = 1; i < MAX_SHARED_X; ++i) o.proj += i < args->m.n && xb >= args->m.xb_first[i];
        o.d_out = args->m.d_out[o.proj];
        o.o0 = (xb - args->m.xb_first[o.proj]) * (RB * 16);
        o.t0 = gm.y;
        o.ge = gm.z;
        o.r = more && gm.x >= 0 ? min(r_stack, gm.w) : 0;
        o.kept = 0;
        o.B = args->m.B_stack[o.proj] + ((int64_t)max(gm.x, 0) * o.d_out + o.o0) * ldb;
        return o;
    };
    // Lane i of instruction j takes chunk i % CPR of row j * (64 / CPR) + i / CPR.  Chunks past the expert's rank are
    // not read (the row's first one is, and masked); without an adapter nothing is but one chunk.
    auto issue_rows = [&](const Item &o, uint4(&rb)[RB * KS]) __attribute__((always_inline)) {
        const int lane = opaque(lane_id);
        const int c = lane % CPR;
        const uint32_t cc = c * 8 < o.r && !o.kept ? (uint32_t)c * 16u : 0u;
        const int rows = o.r > 0 && !o.kept ? o.d_out - o.o0 : 0;
#pragma unroll
        for (int j = 0; j < RB * KS; ++j) {
            const int row = j * (64 / CPR) + lane / CPR;
            rb[j] = ldg_nt(o.B + ((row < rows ? (uint32_t)row * ldb : 0u) + cc));
        }
    };
    Item cur = advance();
    i32x16_t toks = sload_x16(tok_sorted + cur.t0);   // (entries past the record's end: read, not used)
    auto step = [&](uint4(&rb)[RB * KS], uint4(&rb_next)[RB * KS]) __attribute__((always_inline)) {
        const int lane = opaque(lane_id), kq = (lane >> 4) * 8;
        const int pos = cur.t0 + (lane & 15);
        const bool tvalid = pos < cur.ge;
        const int ps = tvalid ? pos : cur.t0;
        const int tok = tvalid ? pick16(toks, lane) : toks[0];
        // lane holds y[token = lane % 16][o0 + b * 16 + 4 * (lane / 16) + i]; rows past d_out read (and never store)
        // the last valid group of four
        f32x4_t part[RB][NSPLIT];
        const int splits = MIXED ? args->m.k_splits[cur.proj] : NSPLIT;   // the projection's own number of parts
        uint4 h[KS], l[KS];
        {
            const int64_t plane = T * (int64_t)cur.d_out;
            const float *ybase = args->m.ybase[cur.proj] + (int64_t)(BY_POS ? ps : tok) * cur.d_out;
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int sp = 0; sp < NSPLIT; ++sp)
                    part[b][sp] = *reinterpret_cast<const f32x4_t *>(
                        ybase + (sp < splits ? sp * plane : 0) + min(cur.o0 + b * 16 + 4 * (lane >> 4), cur.d_out - 4));
            const char *uh = args->m.ug_hi[cur.proj] + (int64_t)ps * ldb, *ul = args->m.ug_lo[cur.proj] + (int64_t)ps * ldb;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                h[ks] = ldg_raw(uh, ks * 32 + kq, cur.r);
                l[ks] = ldg_raw(ul, ks * 32 + kq, cur.r);
            }
        }
        Item nxt = cur;
        if (cur.t0 + 16 < cur.ge) nxt.t0 += 16, nxt.kept = 1;   // a record of several blocks
        else nxt = advance();
        toks = sload_x16(tok_sorted + nxt.t0);
        __builtin_amdgcn_sched_barrier(0);
        issue_rows(nxt, rb_next);
        __builtin_amdgcn_sched_barrier(0);
        // chunk c of row i stands at place c ^ (i / (rows per 256 bytes)): no bank is met twice
        if (!cur.kept) {
#pragma unroll
            for (int j = 0; j < RB * KS; ++j) {
                const int row = j * (64 / CPR) + lane / CPR;
                *reinterpret_cast<uint4 *>(mine + (row * CPR + ((lane % CPR) ^ ((row / (16 / CPR)) & (CPR - 1)))) * 16) =
                    rb[j];
            }
        }
        f32x4_t acc[RB];
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            acc[b] = part[b][0];   // parts are added in order: repeatable
#pragma unroll
            for (int sp = 1; sp < NSPLIT; ++sp)
                if (sp < splits) acc[b] += part[b][sp];
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int k = ks * 32 + kq;   // (past the rank, or without an adapter: zeros)
            const bf16x8_t fh = frag_of(h[ks], k, cur.r), fl = frag_of(l[ks], k, cur.r);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const int row = b * 16 + (lane & 15);
                const int ch = (ks * 4 + (lane >> 4)) ^ ((row / (16 / CPR)) & (CPR - 1));
                const bf16x8_t fa = frag_of(*reinterpret_cast<const uint4 *>(mine + (row * CPR + ch) * 16), k, cur.r);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fh, acc[b], 0, 0, 0);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fl, acc[b], 0, 0, 0);
            }
        }
        char *y = args->m.y[cur.proj];
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int oo = cur.o0 + b * 16 + 4 * (lane >> 4);
            if (tvalid && oo < cur.d_out) store_out(y, cur.d_out, y_f32, tok, oo, acc[b]);   // d_out % 4 == 0
        }
        __builtin_amdgcn_sched_barrier(0);
        cur = nxt;
    };
    uint4 rb0[RB * KS], rb1[RB * KS];
    issue_rows(cur, rb0);
    for (;;) {
        step(rb0, rb1);
        if (!more) return;
        step(rb1, rb0);
        if (!more) return;
    }
}

template <int KS, int NSPLIT, bool BY_POS, int RB, bool MIXED>
__global__ __launch_bounds__(EXPAND_WAVES * 64, expand_stream_wgs(KS, NSPLIT, RB)) void decode_expand_stream_kernel(ExpandStreamArgs)
{
    extern __shared__ __align__(16) char smem[];
    const MOIN_CONST_AS ExpandStreamArgs *args = kernel_args<ExpandStreamArgs>();
    const int P = (int)gridDim.x * EXPAND_WAVES, w = (int)blockIdx.x * EXPAND_WAVES + uniform((int)threadIdx.x >> 6);
    const FirstRecord fr = first_record(args->p.n_groups, args->p.grp_meta, min(w / args->n_xb, args->max_groups - 1));
    if (fr.recs.y > 0) {
        // (the waves that find no item among the others' first)
        const int busy = (fr.recs.x - fr.recs.y) * args->n_xb % P;
        write_base_only<NSPLIT, BY_POS, MIXED>(args, fr.recs.y, w >= busy ? w - busy : w - busy + P, P);
    }
    expand_stream<KS, NSPLIT, BY_POS, RB, MIXED>(args, smem, fr);
}

static ShrinkDParams shrink_params(const PlanView &pv, const DecodeArgs &d)
{
    const LinearArgs &a = d.lin;
    ShrinkDParams p;
    p.x = (const char *)a.x; p.A_stack = (const char *)a.A_stack;
    p.ug_hi = (char *)d.ug_hi; p.ug_lo = (char *)d.ug_lo;
    p.tok_sorted = pv.tok_sorted; p.grp_meta = pv.grp_meta; p.n_groups = pv.n_groups;
    p.d_in = a.d_in; p.r = a.r; p.scale = a.scale; p.act = a.act;
    return p;
}

static DecodeMore decode_more(const DecodeArgs *d, int n);

constexpr int HELD_WGS = 16;            // workgroups per compute unit of the held kernels, at most: a few rounds each
// Tiles keep one block in flight instead of three where the adapters' stream outlasts them (bytes of A_e, if every
// sequence has its own expert): tiles that ask for more only hold it up.  Us of a call, one / three, 300 experts: 256
// tokens, q, k, v at rank 128 (402 MB) 52.8 / 55.0, gate + up at rank 64 (134 MB) 65.5 / 68.0; 512 tokens, q, k, v at rank
// 32 (118 MB) 38.6 / 40.2, rank 128 79.2 / 83.8.  With shorter adapters or fewer of them the launch waits for the tiles'
// own chain of trips to memory (256 tokens, gate + up, rank 32, 67 MB, 60.0 / 56.2; down, rank 16, 46 MB, 39.1 / 33.8),
// and so it does with fewer tokens, whose experts repeat less than the bound says (200 tokens, down, rank 64, 144 MB
// 45.1 / 42.0; 33 tokens, rank 16 31.5 / 25.2).
constexpr int PACED_MIN_T = 256;
constexpr int64_t PACED_MIN_BYTES = 96 << 20;
// Shrink items that a base tile of 32 blocks stands for (one step each; an item of b steps counts as (b + 1) / 2, its
// steps overlap).  q, k, v and down of 256 single tokens: 46 and 49 us counting 1, 44 and 49 with 3, 39 and 41 with 6,
// 40 and 43 with 8.
constexpr int DECODE_TILE_ITEMS = 6;

// Workgroups of a persistent launch: what the chip holds at a time, a multiple of 8 (the XCDs), and no more than
// there can be items.
static int persistent_grid(int per_cu, int64_t items)
{
    const int64_t P = (int64_t)per_cu * compute_units();
    return (int)((std::min(P, std::max<int64_t>(items, 1)) + 7) & ~7LL);
}

// Records tend to span several blocks of 16 tokens (4 tokens per possible group on average is where holding a slab
// in registers for all of a record's blocks began to pay on the 5632-wide projection).
static bool several_blocks(const PlanView &pv)
{
    return pv.chunk > GROUP_CHUNK_MIN && pv.T >= 4 * std::min<int64_t>(pv.S, (int64_t)pv.E + 1);
}

hipError_t launch_decode_shrink(const PlanView &pv, const DecodeArgs &d, hipStream_t stream)
{
    const LinearArgs &a = d.lin;
    if (a.r <= 0 || pv.max_groups <= 0) return hipSuccess;
    const int n_slabs = (a.r + 15) / 16;
    const int64_t items = (int64_t)n_slabs * pv.max_groups;
    if (items > 0x3fffffffLL) return hipErrorInvalidValue;
    // k-steps of 32 per wave
    const int per = ((a.d_in + 31) / 32 + SHRINK_WAVES - 1) / SHRINK_WAVES;
    const ShrinkDParams p = shrink_params(pv, d);
    const dim3 block(SHRINK_WAVES * 64);
    if (several_blocks(pv) && per <= 8) {
        hipLaunchKernelGGL(decode_shrink_kernel<8>, dim3(persistent_grid(HELD_WGS, items)), block, 0, stream, p, n_slabs);
    } else if (several_blocks(pv) && per <= 24) {
        hipLaunchKernelGGL(decode_shrink_kernel<24>, dim3(persistent_grid(HELD_WGS, items)), block, 0, stream, p, n_slabs);
    } else {
        const Turns turns{persistent_grid(2, items), 0, 1};
        hipLaunchKernelGGL((decode_base_shrink_kernel<false, false>), dim3(turns.P), block, STREAM_SMEM, stream,
                           ShrinkStreamArgs{p, LinearKParams{}, decode_more(&d, 1), turns, 0, n_slabs, pv.max_groups});
    }
    return hipGetLastError();
}

bool decode_base_shrink_fits(const PlanView &pv, const DecodeArgs &d)
{
    if (d.lin.r <= 0 || pv.max_groups <= 0 || pv.T <= 0) return false;
    const DecodeBaseShape sh = decode_base_shape(pv.T, d.lin.d_in, d.lin.d_out);
    return sh.dma || sh.slab_blocks > 0;
}

template <class K>
static hipError_t allow_lds(K kern, int bytes)
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

hipError_t prepare_decode_kernels()
{
    hipError_t e = allow_lds(&decode_base_shrink_kernel<true, false>, STREAM_SMEM);
    if (e == hipSuccess) e = allow_lds(&decode_base_shrink_kernel<true, true>, STREAM_SMEM);
    if (e == hipSuccess) e = allow_lds(&decode_base_shrink_kernel<false, false>, STREAM_SMEM);
    return e;
}

// True when the n projections of a call that share x can share its two launches: the same input, contraction length,
// rank, scale, activation, output type and -- those whose base product is cut into tiles, beyond MIX_MAX_T tokens -- number
// of its parts.  (Up to there the parts go by the projection's width: linear.hip's rule for few tokens.)
constexpr int MIX_MAX_T = 128;
static_assert(MIX_MAX_T <= DECODE_MAX_T, "records of 16 tokens, which the streaming expand takes");
bool decode_shared_fits(const PlanView &pv, const DecodeArgs *d, int n)
{
    if (n < 1 || n > MAX_SHARED_X) return false;
    int tile_splits = 0;
    for (int i = 0; i < n; ++i) {
        if (!decode_base_shrink_fits(pv, d[i])) return false;
        const LinearArgs &a = d[i].lin, &a0 = d[0].lin;
        if (decode_base_shape(pv.T, a.d_in, a.d_out).slab_blocks == 0) {
            if (tile_splits != 0 && d[i].k_splits != tile_splits && pv.T > MIX_MAX_T) return false;
            tile_splits = d[i].k_splits;
        }
        if (a.x != a0.x || a.d_in != a0.d_in || a.r != a0.r || a.scale != a0.scale || a.act != a0.act ||
            a.y_f32 != a0.y_f32 || d[i].ybase_by_pos != d[0].ybase_by_pos)
            return false;
    }
    return true;
}

static DecodeMore decode_more(const DecodeArgs *d, int n)
{
    DecodeMore m;
    m.n = n;
    for (int i = 0; i < MAX_SHARED_X; ++i) {
        const DecodeArgs &q = d[i < n ? i : 0];
        m.tile_first[i] = m.slab_first[i] = m.xb_first[i] = 0;
        m.k_splits[i] = q.k_splits;
        m.W[i] = (const char *)q.lin.W; m.A_stack[i] = (const char *)q.lin.A_stack;
        m.B_stack[i] = (const char *)q.lin.B_stack;
        m.ug_hi[i] = (char *)q.ug_hi; m.ug_lo[i] = (char *)q.ug_lo; m.y[i] = (char *)q.lin.y;
        m.ybase[i] = q.ybase;
        m.d_out[i] = q.lin.d_out; m.n_tiles_n[i] = 0;
    }
    return m;
}

hipError_t launch_decode_base_shrink_shared(const PlanView &pv, const DecodeArgs *d, int n, hipStream_t stream)
{
    if (!decode_shared_fits(pv, d, n)) return hipErrorInvalidValue;
    const LinearArgs &a = d[0].lin;
    DecodeMore m = decode_more(d, n);
    int64_t n_tiles = 0, n_w = 0;
    LinearKParams lp{};
    int tile_blocks = 0;   // of a tile's part of the contraction, at most
    for (int i = 0; i < n; ++i) {
        const DecodeBaseShape sh = decode_base_shape(pv.T, a.d_in, d[i].lin.d_out);
        if (!(sh.dma || sh.slab_blocks) || sh.k_splits != d[i].k_splits) return hipErrorInvalidValue;
        m.tile_first[i] = (int)n_tiles;
        m.slab_first[i] = (int)n_w;
        m.n_tiles_n[i] = sh.n_tiles_n;
        if (sh.slab_blocks > 0) {
            n_w += sh.grid;
        } else {
            n_tiles += sh.grid;   // (a multiple of 8, every projection's tiles keep their place in the XCD rotation)
            if (sh.kb_per_split != (a.d_in / CfgDecodeBase::BK + sh.k_splits - 1) / sh.k_splits) return hipErrorInvalidValue;
            tile_blocks = std::max(tile_blocks, sh.kb_per_split);
        }
        if (i == 0 || sh.slab_blocks == 0)   // (what the slabs need of it is the batch's size)
            lp = decode_base_params(pv, a, d[i].ybase, 1, sh, pv.tok_sorted);   // rows in by-expert order
    }
    const int n_slabs = (a.r + 15) / 16;
    const int64_t items = n_w + (int64_t)n_slabs * pv.max_groups * n;
    if (n_tiles + items > 0x3fffffffLL) return hipErrorInvalidValue;
    const ShrinkDParams sp = shrink_params(pv, d[0]);
    const dim3 block(SHRINK_WAVES * 64);
    Turns turns{persistent_grid(2, n_tiles + items), (int)n_tiles, 1};
    if (n_tiles > 0) {
        const int batches = (a.d_in * 2 + SHRINK_WAVES * STREAM_COL - 1) / (SHRINK_WAVES * STREAM_COL);
        const int64_t bytes = (int64_t)std::min(pv.S, pv.E) * a.r * n * a.d_in * 2;
        turns.c = std::max(1, DECODE_TILE_ITEMS * tile_blocks / (16 * (batches + 1)));
        if (pv.T >= PACED_MIN_T && bytes > PACED_MIN_BYTES)
            hipLaunchKernelGGL((decode_base_shrink_kernel<true, true>), dim3(turns.P), block, STREAM_SMEM, stream,
                               ShrinkStreamArgs{sp, lp, m, turns, (int)n_w, n_slabs, pv.max_groups});
        else
            hipLaunchKernelGGL((decode_base_shrink_kernel<true, false>), dim3(turns.P), block, STREAM_SMEM, stream,
                               ShrinkStreamArgs{sp, lp, m, turns, (int)n_w, n_slabs, pv.max_groups});
    } else {
        hipLaunchKernelGGL((decode_base_shrink_kernel<false, false>), dim3(turns.P), block, STREAM_SMEM, stream,
                           ShrinkStreamArgs{sp, lp, m, turns, (int)n_w, n_slabs, pv.max_groups});
    }
    return hipGetLastError();
}

hipError_t launch_decode_base_shrink(const PlanView &pv, const DecodeArgs &d, hipStream_t stream)
{
    return launch_decode_base_shrink_shared(pv, &d, 1, stream);
}

hipError_t launch_decode_expand_shared(const PlanView &pv, const DecodeArgs *d, int n, hipStream_t stream)
{
    if (n < 1 || n > MAX_SHARED_X) return hipErrorInvalidValue;
    if (pv.max_groups <= 0) return hipSuccess;
    const LinearArgs &a = d[0].lin;
    int k_splits = d[0].k_splits;   // of the kernel; a projection with fewer parts adds its own
    for (int i = 1; i < n; ++i) {
        if (d[i].lin.r != a.r || d[i].lin.y_f32 != a.y_f32 || d[i].ybase_by_pos != d[0].ybase_by_pos)
            return hipErrorInvalidValue;
        k_splits = std::max(k_splits, d[i].k_splits);
    }
    ExpandKParams p;
    p.B_stack = (const char *)a.B_stack; p.ug_hi = (const char *)d[0].ug_hi; p.ug_lo = (const char *)d[0].ug_lo;
    p.ybase = d[0].ybase; p.y = (char *)a.y;
    p.tok_sorted = pv.tok_sorted; p.grp_meta = pv.grp_meta; p.n_groups = pv.n_groups;
    p.T = pv.T; p.d_out = a.d_out; p.r = a.r; p.k_splits = d[0].k_splits; p.y_f32 = a.y_f32;
    const int nks = (a.r + 31) / 32;
    const bool streams = nks <= 4 && !several_blocks(pv);
    constexpr int RB = 4;   // 16-row blocks per wave of the held form
    const bool large = pv.T > DECODE_MAX_T && k_splits == 1 && !d[0].ybase_by_pos;
    const int ks = nks <= 2 ? nks : 4, stream_rb = expand_stream_rb(ks, large);
    const int rows = streams ? stream_rb * 16 : EXPAND_WAVES * RB * 16;
    DecodeMore m = decode_more(d, n);
    int64_t xb = 0, base_only = 0;
    for (int i = 0; i < n; ++i) {
        m.xb_first[i] = (int)xb;
        xb += (d[i].lin.d_out + rows - 1) / rows;
        base_only += pv.T * ((d[i].lin.d_out + BASE_ONLY_COLS - 1) / BASE_ONLY_COLS);
    }
    const int64_t items = xb * pv.max_groups;
    if (items > 0x3fffffffLL) return hipErrorInvalidValue;
    // (a wave per item, or per piece of a base-only token, as far as the chip holds them)
    const int64_t stream_wgs = (std::max(items, base_only) + EXPAND_WAVES - 1) / EXPAND_WAVES;
    const dim3 grid((unsigned)(streams ? persistent_grid(expand_stream_wgs(ks, k_splits, stream_rb), stream_wgs)
                                       : persistent_grid(HELD_WGS, items)));
    // parts that differ: slabs (one) beside tiles, or tiles of up to MIX_MAX_T tokens (decode_shared_fits)
    bool mixed = false;
    for (int i = 1; i < n; ++i) mixed = mixed || d[i].k_splits != d[0].k_splits;
    if (mixed && (!d[0].ybase_by_pos || pv.T > MIX_MAX_T || (nks <= 4 && !streams))) return hipErrorInvalidValue;
#define MOIN_EXPAND_STREAM(KS, NS, BP, SRB, MIX)                                                                          \
    hipLaunchKernelGGL((decode_expand_stream_kernel<(KS > 0 ? KS : 1), NS, BP, SRB, MIX>), grid, dim3(EXPAND_WAVES * 64), \
                       EXPAND_WAVES * expand_stage(KS, SRB), stream, ExpandStreamArgs{p, m, (int)xb, pv.max_groups})
#define MOIN_EXPAND_HELD(KS, NS, BP, MIX)                                                                               \
    hipLaunchKernelGGL((decode_expand_kernel<KS, NS, BP, RB, MIX>), grid, dim3(EXPAND_WAVES * 64), 0, stream, p, m, (int)xb)
#define MOIN_EXPAND_R(KS, NS, BP)                                                                                      \
    do {                                                                                                               \
        constexpr bool may_mix = NS >= 2 && BP;                                                                        \
        if (KS > 0 && streams && NS == 1 && !BP && large) MOIN_EXPAND_STREAM(KS, 1, false, 4, false);                  \
        else if (KS > 0 && streams && mixed) MOIN_EXPAND_STREAM(KS, NS, BP, (expand_stream_rb(KS, false)), may_mix);   \
        else if (KS > 0 && streams) MOIN_EXPAND_STREAM(KS, NS, BP, (expand_stream_rb(KS, false)), false);              \
        else if (mixed) MOIN_EXPAND_HELD(KS, NS, BP, (KS == 0 && may_mix)); /* (a small batch streams) */             \
        else MOIN_EXPAND_HELD(KS, NS, BP, false);                                                                      \
    } while (0)
#define MOIN_EXPAND_S(KS, NS)                                                                                  \
    do {                                                                                                       \
        if (d[0].ybase_by_pos) MOIN_EXPAND_R(KS, NS, true);                                                    \
        else MOIN_EXPAND_R(KS, NS, false);                                                                     \
    } while (0)
#define MOIN_EXPAND(KS)                                  \
    switch (k_splits) {                                  \
    case 1: MOIN_EXPAND_S(KS, 1); break;                 \
    case 2: MOIN_EXPAND_S(KS, 2); break;                 \
    case 3: MOIN_EXPAND_S(KS, 3); break;                 \
    case 4: MOIN_EXPAND_S(KS, 4); break;                 \
    default: return hipErrorInvalidValue;                \
    }
    if (nks <= 1) MOIN_EXPAND(1)
    else if (nks <= 2) MOIN_EXPAND(2)
    else if (nks <= 4) MOIN_EXPAND(4)
    else MOIN_EXPAND(0)
#undef MOIN_EXPAND
#undef MOIN_EXPAND_S
#undef MOIN_EXPAND_R
#undef MOIN_EXPAND_HELD
#undef MOIN_EXPAND_STREAM
    return hipGetLastError();
}

hipError_t launch_decode_expand(const PlanView &pv, const DecodeArgs &d, hipStream_t stream)
{
    return launch_decode_expand_shared(pv, &d, 1, stream);
}

}  // namespace moin
