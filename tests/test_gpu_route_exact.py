"""The routes that compute squared distances themselves (fp32 moin_route, moin_route_topk): the kernel that takes
every pair, and the screened search, whose answer has to be that of the exhaustive one bit for bit."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc
from tests.test_gpu_route_topk import _check as check_topk

pytestmark = pytest.mark.gpu


def _inputs(N, K, D, dtype, kind, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    cent = torch.randn((K, D), device="cuda", generator=g)
    emb = torch.randn((N, D), device="cuda", generator=g)
    if kind == "offset":        # a large common part: the screened scores cancel, many groups stay candidates
        cent, emb = cent + 30.0, emb + 30.0
    elif kind == "near":        # tight clusters and exact duplicates
        cent = cent[torch.arange(K, device="cuda") % 50] + 1e-3 * cent
        cent[K // 2:K // 2 + 5] = cent[3]
        emb = cent[torch.arange(N, device="cuda") * 7 % K] + 1e-3 * emb
    elif kind == "odd":         # values beyond the bound's reach, and not-a-numbers
        cent[5, 1], cent[9, 0], emb[3, 2], emb[7, 0] = float("nan"), 3e38, float("nan"), 3e38
    return emb.to(dtype), cent.to(dtype)


@pytest.mark.parametrize("N,K,D", [(1, 1, 4), (1, 8, 8), (8, 7, 252), (9, 9, 256), (65, 33, 260), (7, 500, 384),
                                   (4096, 17, 64), (4097, 20, 12), (300, 64, 1024)])
def test_direct_fp32_router_edges(N, K, D):
    emb, cent = _inputs(N, K, D, torch.float32, "plain", N + K + D)
    print(f"[gpu] direct fp32 router N={N} K={K} D={D}", flush=True)
    slot = torch.from_numpy(wl.retained_slot_table(K, max(1, K - 3), seed=K)).cuda()
    for kw, el in ((dict(), None), (dict(slot_of_centroid=slot, retained_only=True), slot.cpu().numpy() >= 0)):
        for _ in range(2):      # twice: the scratch cleans itself
            eids, cids, counts = moin.moin_route(gc.ctx(), emb, cent, want_counts=True, **kw)
            gc.ctx().check()
            gc.check_route(emb, cent, cids, eligible=el)
            assert torch.equal(counts.long(), torch.bincount(cids.long(), minlength=K))
            assert torch.equal(eids, cids if el is None else slot[cids.long()])


# sizes past the line where screening begins (150 M pair-dimensions), ragged in every direction
@pytest.mark.parametrize("kind", ["plain", "offset", "near", "odd"])
@pytest.mark.parametrize("N,K,D", [(1001, 700, 260), (130, 5000, 384), (5001, 257, 132)])
def test_screened_fp32_router_equals_the_exhaustive_one(N, K, D, kind):
    emb, cent = _inputs(N, K, D, torch.float32, kind, 3 * N + K + D)
    print(f"[gpu] screened fp32 router N={N} K={K} D={D} {kind}", flush=True)
    slot = torch.from_numpy(wl.retained_slot_table(K, K - 100, seed=K)).cuda()
    for kw in (dict(), dict(slot_of_centroid=slot, retained_only=True)):
        got = moin.moin_route(gc.ctx(), emb, cent, want_counts=True, **kw)
        ref = moin.moin_route(gc.ctx(), emb, cent, want_counts=True, static=True, **kw)   # allocates nothing: every pair
        gc.ctx().check()
        for a, b in zip(got, ref):
            assert torch.equal(a, b)
    if kind in ("plain", "near"):
        gc.check_route(emb, cent, moin.moin_route(gc.ctx(), emb, cent)[1], sample=np.arange(0, N, 11))


# the screen's blocks of 32 values and their remainders: one row's end on both sides of a block and of a padded pair
@pytest.mark.parametrize("N,K,D", [(2100, 2201, 36), (1500, 1601, 64), (2600, 1001, 68), (2000, 801, 96), (2000, 801, 100)])
def test_screened_blocks_of_high_parts_and_remainders(N, K, D):
    emb, cent = _inputs(N, K, D, torch.float32, "near", N + K + D)
    print(f"[gpu] screened fp32 router N={N} K={K} D={D}", flush=True)
    got = moin.moin_route(gc.ctx(), emb, cent, want_counts=True)
    ref = moin.moin_route(gc.ctx(), emb, cent, want_counts=True, static=True)   # every pair
    gc.ctx().check()
    for a, b in zip(got, ref):
        assert torch.equal(a, b)


@pytest.mark.parametrize("kind", ["plain", "offset", "near", "odd"])
@pytest.mark.parametrize("dtype,D", [(torch.float32, 260), (torch.bfloat16, 264), (torch.bfloat16, 256)])
def test_screened_topk_equals_the_exhaustive_one(dtype, D, kind):
    N, K = 1030, 611
    emb, cent = _inputs(N, K, D, dtype, kind, 17 + D)
    slot = torch.from_numpy(wl.retained_slot_table(K, K - 100, seed=K)).cuda()
    for k, kw in ((1, dict()), (3, dict(slot_of_centroid=slot, retained_only=True)), (8, dict())):
        print(f"[gpu] screened topk k={k} D={D} {dtype} {kind}", flush=True)
        whole = moin.moin_route_topk(gc.ctx(), emb, cent, k, **kw)
        # a few queries at a time stay below the line: every distance computed
        parts = [moin.moin_route_topk(gc.ctx(), emb[i:i + 206], cent, k, **kw) for i in range(0, N, 206)]
        gc.ctx().check()
        for a, b in zip(whole, (torch.cat(t) for t in zip(*parts))):
            assert torch.equal(a, b)
    if kind != "odd":
        check_topk(emb[:60].contiguous(), cent, 8, what=kind)


def test_a_small_fp32_call_leaves_the_norms_kept_for_bf16_alone():
    # a server that routes bf16 requests against one table and, in between, tallies fp32 queries against another:
    # the second call's scratch must not reach the norms that MOIN_ROUTE_SAME_CENTROIDS lets the third one reuse
    ctx = moin.Context(0)
    try:
        emb, cent = _inputs(64, 5000, 64, torch.bfloat16, "plain", 3)
        small, table = _inputs(1000, 500, 16, torch.float32, "plain", 4)
        print("[gpu] bf16 norms kept across a small fp32 call", flush=True)
        first = moin.moin_route(ctx, emb, cent, want_counts=True)
        _, none, counts = moin.moin_route(ctx, small, table, want_centroid_ids=False, want_counts=True)
        again = moin.moin_route(ctx, emb, cent, want_counts=True, same_centroids=True)
        ctx.check()
        assert none is None and int(counts.sum()) == 1000
        for a, b in zip(first, again):
            assert torch.equal(a, b)
    finally:
        ctx.close()


def test_searches_whose_copies_do_not_fit_answer_without_them():
    # the screened and the padded search copy the table; with less than that left on the device the search that
    # needs no copy gives the same answer
    f32, bf16 = torch.float32, torch.bfloat16
    shapes = {f32: (600_000, 1024), bf16: (1_200_000, 1032)}     # 2.4 GB, and as much again copied
    g = torch.Generator(device="cuda").manual_seed(12)
    tables, picks = {}, {}
    for dtype, (K, D) in shapes.items():
        cent = torch.empty((K, D), dtype=dtype, device="cuda").normal_(generator=g)
        picks[dtype] = torch.arange(8, device="cuda") * (K // 8) + 3
        emb = cent[picks[dtype]].float() + 0.1 * torch.randn((8, D), device="cuda", generator=g)
        tables[dtype] = (emb.to(dtype), cent)

    def run(dtype, topk):
        ctx = moin.Context(0)
        try:
            out = moin.moin_route_topk(ctx, *tables[dtype], 2) if topk else moin.moin_route(ctx, *tables[dtype])[:2]
            ctx.check()
            return out, ctx.workspace_bytes()
        finally:
            ctx.close()

    cases = ((f32, True), (f32, False), (bf16, False))
    print("[gpu] searches with their copies", flush=True)
    want = [run(*c) for c in cases]
    torch.cuda.empty_cache()
    rest = torch.empty(torch.cuda.mem_get_info()[0] - (1 << 30), dtype=torch.uint8, device="cuda")
    try:
        print("[gpu] and without", flush=True)
        got = [run(*c) for c in cases]
    finally:
        del rest
        torch.cuda.empty_cache()
    for (dtype, _), (a, ua), (b, ub) in zip(cases, want, got):
        assert ua > 2 << 30 > 1 << 30 > ub
        assert torch.equal(a[1].reshape(8, -1)[:, 0].long(), picks[dtype])
        for x, y in zip(a, b):
            assert torch.equal(x, y)


def test_screened_parts_of_long_rows_stay_small():
    # the planes of the queries are written for a part of the batch at a time, whatever the rows' length
    emb, cent = _inputs(20001, 300, 4096, torch.float32, "near", 5)
    ctx = moin.Context(0)
    try:
        print("[gpu] screened fp32 router, long rows", flush=True)
        got = moin.moin_route(ctx, emb, cent, want_counts=True)
        ref = moin.moin_route(ctx, emb, cent, want_counts=True, static=True)
        ctx.check()
        for a, b in zip(got, ref):
            assert torch.equal(a, b)
        assert ctx.workspace_bytes() <= 256 << 20
    finally:
        ctx.close()
