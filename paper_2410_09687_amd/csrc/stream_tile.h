// What the streaming prefill kernels know of a call and of a tile.
#pragma once
#include "gemm_core.h"
#include "kernels.h"

namespace moin {

// The halves of a call's plan tiles (TILE_M / 2 tokens each) that hold any tokens, numbered without the others: a workgroup that
// has nothing to do still takes its turn, and the ones behind it may have to wait for a compute unit that is busy although another
// is free.  (1700 tokens in eight sequences of 75 to 310, three times 2048 -> 1024, 360 halves of 528: eight
// workgroups started 25 us late, 44 us instead of 30.)
struct HalfTiles {
    static constexpr int CHUNKS = 4;           // beyond 64 * CHUNKS plan tiles the empty halves are numbered too
    unsigned long long second[CHUNKS];         // which plan tiles have tokens in their second half
    int n_tiles, count;

    __device__ __forceinline__ HalfTiles(const int *tile_rows, const int *n_tiles_, int max_tiles)
    {
        const int lane = threadIdx.x & 63;
        const int first = lane < max_tiles ? tile_rows[lane] : 0;   // (under way with the number of tiles)
        n_tiles = uniform(*n_tiles_);
        second[0] = __ballot(lane < n_tiles && first > TILE_M / 2);
        count = n_tiles + __popcll(second[0]);
        if (n_tiles <= 64) return;
#pragma unroll
        for (int i = 1; i < CHUNKS; ++i) {
            const int rows = i * 64 + lane < min(n_tiles, max_tiles) ? tile_rows[i * 64 + lane] : 0;
            second[i] = __ballot(rows > TILE_M / 2);
            count += __popcll(second[i]);
        }
        if (n_tiles > 64 * CHUNKS) count = 2 * n_tiles;
    }
    // Half number j (< count): its plan tile times two, plus one for a second half.
    __device__ __forceinline__ int find(int j) const
    {
        if (n_tiles > 64 * CHUNKS) return j;
        if (n_tiles <= 64) return find_in(0, j);
        int at = 0;
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int halves = min(max(n_tiles - i * 64, 0), 64) + __popcll(second[i]);
            if (j >= 0 && j < halves) at = find_in(i, j);
            j -= halves;
        }
        return at;
    }

private:
    __device__ __forceinline__ int find_in(int i, int j) const   // j: counted from the chunk's first half
    {
        const int lane = threadIdx.x & 63;
        auto before = [&](int t) { return t + __popcll(second[i] & ((1ull << t) - 1)); };   // halves of the chunk's first t tiles
        const int t = __popcll(__ballot(i * 64 + lane < n_tiles && before(lane) <= j)) - 1;
        return uniform((i * 64 + t) * 2 + j - before(t));
    }
};

// The same with quarters of plan tiles, of calls of at most MAX plan tiles.
struct QuarterTiles {
    static constexpr int MAX = 64;
    unsigned long long more[3];   // which plan tiles have tokens in their second, third, fourth quarter
    int n_tiles, count;

    __device__ __forceinline__ QuarterTiles(const int *tile_rows, const int *n_tiles_, int max_tiles)
    {
        const int lane = threadIdx.x & 63;
        const int rows = lane < max_tiles ? tile_rows[lane] : 0;   // (under way with the number of tiles)
        n_tiles = min(uniform(*n_tiles_), MAX);
        count = n_tiles;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            more[q] = __ballot(lane < n_tiles && rows > (q + 1) * (TILE_M / 4));
            count += __popcll(more[q]);
        }
    }
    // Quarter number j (< count): its plan tile times four, plus its place there.
    __device__ __forceinline__ int find(int j) const
    {
        const int lane = threadIdx.x & 63;
        auto before = [&](int t) {   // quarters of the first t tiles
            const unsigned long long m = (1ull << t) - 1;
            return t + __popcll(more[0] & m) + __popcll(more[1] & m) + __popcll(more[2] & m);
        };
        const int t = __popcll(__ballot(lane < n_tiles && before(lane) <= j)) - 1;
        return uniform(t * 4 + j - before(t));
    }
};

namespace stream {

constexpr int BK = 64;          // contraction steps of a block
constexpr int ROWB = BK * 2;    // LDS row pitch

// Up to MAX_SHARED_X projections that read the same x (q, k, v; gate, up) in one launch: the column
// tiles of projection i follow those of projection i - 1, so a narrow projection's tiles (k, v: one
// column of tiles) ride in the wide one's stream and share its x panels in L2.
struct Params {
    const char *x;
    const char *W[MAX_SHARED_X], *B_stack[MAX_SHARED_X], *u_hi[MAX_SHARED_X], *u_lo[MAX_SHARED_X];
    char *y[MAX_SHARED_X];
    int d_out[MAX_SHARED_X];
    int tn_start[MAX_SHARED_X];   // first column tile of each projection (tn_start[0] = 0)
    int n_proj;
    const int *tile_row0, *tile_rows, *tile_expert, *tile_rank, *n_tiles;
    int d_in, r, ldu;             // (ldu: columns of u as stored)
    int n_tiles_n;                // column tiles of all projections together
    int max_tiles;                // entries of the plan's tile arrays
    int y_f32;
    int by_columns;               // linear_mid.hip: tiles of one column are neighbours (else: of one row)
};

// Everything a tile needs, all wave-uniform.
struct Tile {
    const char *q0, *p0;       // x rows / W rows of the tile at k = 0
    const char *uh, *ul, *be;  // adapter operands (aliases of q0 / p0 without adapter)
    int q_rows, p_rows;        // valid tokens (of a plan tile's part: <= 0 where it has none) / outputs
    int rank;                  // columns of u that count (load_tile alone reads it; without it the streaming kernel's registers fall
                               // out otherwise: 270.0 -> 271.4 us for 32 768 tokens 2048 -> 2048 with routing)
    int nkb1;                  // adapter blocks per half (0: no adapter)
    int total;                 // blocks of the tile: those of the base, 2 * nkb1
    int row0, n0;
    char *y;                   // the projection's output and its width
    int d_out;
    int valid;
};

// Tile (tm, tn) of BTP outputs x BTQ tokens; a plan tile is TILE_M / BTQ of them.
template <int BTP, int BTQ>
__device__ __forceinline__ Tile load_tile(const Params &p, int tm, int tn)
{
    Tile t;
    constexpr int SUB = TILE_M / BTQ;
    const int pt = tm / SUB, sub = tm % SUB;
    const int e = uniform(p.tile_expert[pt]);
    t.row0 = uniform(p.tile_row0[pt]) + sub * BTQ;
    t.q_rows = min(BTQ, uniform(p.tile_rows[pt]) - sub * BTQ);
    // the projection of this column tile (picked by comparison, not by indexing: indexing the
    // parameter arrays would put them in scratch)
    const char *W = p.W[0], *B_stack = p.B_stack[0], *u_hi = p.u_hi[0], *u_lo = p.u_lo[0];
    int tn0 = 0;
    t.y = p.y[0];
    t.d_out = p.d_out[0];
#pragma unroll
    for (int i = 1; i < MAX_SHARED_X; ++i)
        if (i < p.n_proj && tn >= p.tn_start[i]) {
            W = p.W[i]; B_stack = p.B_stack[i]; u_hi = p.u_hi[i]; u_lo = p.u_lo[i];
            t.y = p.y[i];
            t.d_out = p.d_out[i];
            tn0 = p.tn_start[i];
        }
    t.n0 = (tn - tn0) * BTP;
    t.p_rows = min(BTP, t.d_out - t.n0);
    const int64_t ldx = (int64_t)p.d_in * 2, ldu = (int64_t)p.ldu * 2, ldb = (int64_t)p.r * 2;
    t.q0 = p.x + (int64_t)t.row0 * ldx;
    t.p0 = W + (int64_t)t.n0 * ldx;
    // adapter blocks up to the expert's own rank (the shrink wrote zeros from there to the block end)
    const int re = min(p.r, uniform(p.tile_rank[pt]));
    const bool lora = e >= 0 && re > 0;
    t.rank = lora ? re : 0;
    t.nkb1 = (t.rank + BK - 1) / BK;
    t.total = (p.d_in + BK - 1) / BK + 2 * t.nkb1;
    t.uh = lora ? u_hi + (int64_t)t.row0 * ldu : t.q0;
    t.ul = lora ? u_lo + (int64_t)t.row0 * ldu : t.q0;
    t.be = lora ? B_stack + ((int64_t)e * t.d_out + t.n0) * ldb : t.p0;
    return t;
}

// Host: the parameters of n projections on column tiles of btp outputs; returns the number of these.
inline int fill_params(Params *p, const PlanView &pv, const LinearArgs *a, int n, int btp)
{
    p->x = (const char *)a[0].x;
    p->n_proj = n;
    int tn = 0;
    for (int i = 0; i < MAX_SHARED_X; ++i) {
        const LinearArgs &ai = a[i < n ? i : 0];
        p->W[i] = (const char *)ai.W; p->B_stack[i] = (const char *)ai.B_stack;
        p->u_hi[i] = (const char *)ai.u_hi; p->u_lo[i] = (const char *)ai.u_lo;
        p->y[i] = (char *)ai.y;
        p->d_out[i] = ai.d_out;
        p->tn_start[i] = tn;
        if (i < n) tn += (ai.d_out + btp - 1) / btp;
    }
    p->tile_row0 = pv.tile_row0; p->tile_rows = pv.tile_rows; p->tile_expert = pv.tile_expert;
    p->tile_rank = pv.tile_rank;
    p->n_tiles = pv.n_tiles;
    p->max_tiles = pv.max_tiles;
    p->d_in = a[0].d_in; p->r = a[0].r; p->ldu = a[0].ldu;
    p->n_tiles_n = tn;
    p->y_f32 = a[0].y_f32;
    p->by_columns = 0;
    return tn;
}

}  // namespace stream

}  // namespace moin
