"""The calls of the hot path can be recorded into a HIP graph (no allocation, no clearing copy, no host
read between their kernels once the workspace has its size) and every replay gives the bits of the eager
call on the inputs then in place."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


def _inputs(name, d_in, d_out, r, E, lens, seed, dist="zipf"):
    w = wl.LinearWorkload(name, d_in, d_out, r, E, lens, dist, 1.1, 2.0, seed=seed)
    return wl.make_linear_inputs(w, "cuda")


def _replay_check(what, inp, call):
    """call(x, eids, out) runs the library on inp's weights; x and eids are overwritten between replays."""
    ctx = gc.ctx()
    g0 = torch.Generator(device="cuda").manual_seed(5)
    xs = [inp.x.clone()] + [torch.randn(inp.x.shape, device="cuda", generator=g0).to(torch.bfloat16)
                            for _ in range(2)]
    ids = [inp.expert_ids.clone(), inp.expert_ids.flip(0).contiguous(),
           torch.where(inp.expert_ids % 3 == 0, torch.full_like(inp.expert_ids, -1), inp.expert_ids)]
    x, eids = inp.x.clone(), inp.expert_ids.clone()
    y_graph = torch.empty((inp.wl.T, inp.wl.d_out), dtype=torch.bfloat16, device="cuda")
    y_eager = torch.empty_like(y_graph)
    print(f"[gpu] graph {what}: eager warm-up (sizes the workspace)", flush=True)
    call(x, eids, y_eager)
    ctx.check()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(x, eids, y_graph)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    print(f"[gpu] graph {what}: capture", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(x, eids, y_graph)
    for rep in range(3):
        print(f"[gpu] graph {what}: replay {rep}", flush=True)
        # the program's own eager work and a synchronisation between the replays
        x.copy_(xs[rep])
        eids.copy_(ids[rep])
        y_graph.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        call(x, eids, y_eager)
        ctx.check()
        assert torch.equal(y_graph.view(torch.int16), y_eager.view(torch.int16)), f"{what}: replay {rep}"
    # and the last replay against the oracle, on the inputs it ran on
    ref = gc.oracle_rows(wl.LinearInputs(inp.wl, x, inp.W, inp.A_stack, inp.B_stack, inp.seq_offsets, eids))
    gc.compare_linear(y_graph, ref, what=f"{what}/graph")


def test_decode_call_replays_from_a_graph():
    inp = _inputs("graph_dec", 512, 520, 64, 40, [1] * 192, seed=71)
    ctx = gc.ctx()
    _replay_check("decode", inp, lambda x, e, out: moin.moin_lora_linear(
        ctx, x, inp.seq_offsets, e, inp.W, inp.A_stack, inp.B_stack, 2.0, out=out))


def test_prefill_call_replays_from_a_graph():
    rng = np.random.default_rng(72)
    inp = _inputs("graph_pre", 256, 264, 64, 6, rng.integers(1, 400, size=12).tolist(), seed=72, dist="uniform")
    assert inp.wl.T > 1024
    ctx = gc.ctx()
    _replay_check("prefill", inp, lambda x, e, out: moin.moin_lora_linear(
        ctx, x, inp.seq_offsets, e, inp.W, inp.A_stack, inp.B_stack, 2.0, out=out))


def test_gathered_batch_call_replays_from_a_graph():
    # more than 1024 tokens in single-token sequences: token grouping, plain-tile base product, gather kernels
    inp = _inputs("graph_gather", 256, 264, 64, 30, [1] * 1500, seed=74)
    ctx = gc.ctx()
    _replay_check("gathered", inp, lambda x, e, out: moin.moin_lora_linear(
        ctx, x, inp.seq_offsets, e, inp.W, inp.A_stack, inp.B_stack, 2.0, out=out))


def test_whole_request_step_replays_from_a_graph():
    # routing + histogram + slot map + grouping in one launch, then the layer: the step a serving loop
    # repeats.  The router's scratch cleans itself, so every replay starts from what the one before left.
    rng = np.random.default_rng(77)
    S, K, D, E = 24, 300, 128, 260
    inp = _inputs("graph_step", 256, 264, 64, E, rng.integers(1, 200, size=S).tolist(), seed=77, dist="uniform")
    rin = wl.make_route_inputs(wl.RouteWorkload("graph_step", S, K, D, "bf16", True, 78), "cuda")
    slots = torch.from_numpy(wl.retained_slot_table(K, E, seed=79)).cuda()
    ctx = gc.ctx()
    emb, x = rin.emb.clone(), inp.x.clone()
    plan_g, plan_e = moin.Plan(ctx), moin.Plan(ctx)
    outs_g = (torch.empty(S, dtype=torch.int32, device="cuda"), None, torch.empty(K, dtype=torch.int32, device="cuda"))
    outs_e = (torch.empty(S, dtype=torch.int32, device="cuda"), None, torch.empty(K, dtype=torch.int32, device="cuda"))
    y_graph = torch.empty((inp.wl.T, inp.wl.d_out), dtype=torch.bfloat16, device="cuda")
    y_eager = torch.empty_like(y_graph)

    def call(plan, outs, y):
        moin.moin_route_plan(ctx, plan, emb, rin.centroids, inp.seq_offsets, inp.wl.T, E, slot_of_centroid=slots,
                             out=outs, same_centroids=True)
        moin.moin_lora_linear_planned(ctx, plan, x, inp.W, inp.A_stack, inp.B_stack, 2.0, out=y)

    print("[gpu] graph step: eager warm-up", flush=True)
    call(plan_e, outs_e, y_eager)
    call(plan_g, outs_g, y_graph)
    ctx.check()
    torch.cuda.synchronize()
    print("[gpu] graph step: capture", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(plan_g, outs_g, y_graph)
    g0 = torch.Generator(device="cuda").manual_seed(8)
    for rep in range(3):
        print(f"[gpu] graph step: replay {rep}", flush=True)
        emb.copy_(rin.centroids[torch.randperm(K, device="cuda", generator=g0)[:S]]
                  + 0.05 * torch.randn((S, D), device="cuda", generator=g0).to(torch.bfloat16))
        x.copy_(torch.randn(x.shape, device="cuda", generator=g0).to(torch.bfloat16))
        y_graph.fill_(float("nan"))
        outs_g[0].fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        call(plan_e, outs_e, y_eager)
        ctx.check()
        assert torch.equal(outs_g[0], outs_e[0]) and torch.equal(outs_g[2], outs_e[2]), f"step replay {rep}: ids"
        assert torch.equal(y_graph.view(torch.int16), y_eager.view(torch.int16)), f"step replay {rep}"
    # the graph's ids are the slot-mapped winners of a plain routing call, which is checked against the oracle
    _, cids, _ = moin.moin_route(ctx, emb, rin.centroids)
    ctx.check()
    gc.check_route(emb, rin.centroids, cids)
    assert torch.equal(outs_g[0], slots[cids.long()])
    ref = gc.oracle_rows(wl.LinearInputs(inp.wl, x, inp.W, inp.A_stack, inp.B_stack, inp.seq_offsets, outs_g[0]))
    gc.compare_linear(y_graph, ref, what="step/graph")
    plan_g.close()
    plan_e.close()


def test_quantised_base_call_replays_from_a_graph():
    rng = np.random.default_rng(73)
    inp = _inputs("graph_mx", 256, 264, 64, 6, rng.integers(1, 400, size=12).tolist(), seed=73, dist="uniform")
    ctx = gc.ctx()
    Wq, Ws = moin.moin_mx_quantize(ctx, inp.W, blocked=True)
    x, eids = inp.x.clone(), inp.expert_ids.clone()
    y_graph = torch.empty((inp.wl.T, inp.wl.d_out), dtype=torch.bfloat16, device="cuda")

    def call(out):
        moin.moin_lora_linear_mx(ctx, x, inp.seq_offsets, eids, Wq, Ws, inp.A_stack, inp.B_stack, 2.0, out=out)

    y_eager = torch.empty_like(y_graph)
    call(y_eager)
    ctx.check()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(y_graph)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(y_graph)
    g0 = torch.Generator(device="cuda").manual_seed(6)
    for rep in range(3):
        print(f"[gpu] graph mx: replay {rep}", flush=True)
        x.copy_(torch.randn(x.shape, device="cuda", generator=g0).to(torch.bfloat16))
        y_graph.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        call(y_eager)
        ctx.check()
        assert torch.equal(y_graph.view(torch.int16), y_eager.view(torch.int16)), f"mx replay {rep}"


def test_two_contexts_on_two_streams_do_not_disturb_each_other():
    # a context owns its workspace and serves one stream at a time: two of them, each on its own stream,
    # with their calls interleaved, give what each gives alone
    a = _inputs("two_ctx_a", 256, 264, 64, 6, [300, 500, 700], seed=75, dist="uniform")
    b = _inputs("two_ctx_b", 384, 136, 128, 9, [1] * 400, seed=76)
    c0 = gc.ctx()
    want_a = moin.moin_lora_linear(c0, a.x, a.seq_offsets, a.expert_ids, a.W, a.A_stack, a.B_stack, 2.0)
    want_b = moin.moin_lora_linear(c0, b.x, b.seq_offsets, b.expert_ids, b.W, b.A_stack, b.B_stack, 2.0)
    c0.check()
    c1, c2 = moin.Context(0), moin.Context(0)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    try:
        for rep in range(4):
            print(f"[gpu] two contexts, round {rep}", flush=True)
            with torch.cuda.stream(s1):
                ya = moin.moin_lora_linear(c1, a.x, a.seq_offsets, a.expert_ids, a.W, a.A_stack, a.B_stack, 2.0)
            with torch.cuda.stream(s2):
                yb = moin.moin_lora_linear(c2, b.x, b.seq_offsets, b.expert_ids, b.W, b.A_stack, b.B_stack, 2.0)
            with torch.cuda.stream(s1):
                ya2 = moin.moin_lora_linear(c1, a.x, a.seq_offsets, a.expert_ids, a.W, a.A_stack, a.B_stack, 2.0)
            s1.synchronize()
            s2.synchronize()
            assert torch.equal(ya, want_a) and torch.equal(ya2, want_a) and torch.equal(yb, want_b)
        with torch.cuda.stream(s1):
            c1.check()
        with torch.cuda.stream(s2):
            c2.check()
    finally:
        torch.cuda.synchronize()
        c1.close()
        c2.close()


def test_capture_refuses_to_grow_and_keeps_what_a_graph_recorded():
    # A fresh context has no workspace: a call on a capturing stream must fail (nothing may be allocated
    # there) and record nothing.  After reserving, the same capture works.  A later eager call with larger
    # shapes replaces workspace and plan buffer, but the blocks the graph recorded stay allocated, so a
    # replay still computes the right thing.
    ctx = moin.Context(0)
    try:
        inp = _inputs("graph_grow", 256, 264, 64, 12, [1] * 96, seed=75)
        big = _inputs("graph_grow_big", 256, 520, 64, 12, [1] * 700, seed=76)
        x, eids = inp.x.clone(), inp.expert_ids.clone()
        y_graph = torch.empty((inp.wl.T, inp.wl.d_out), dtype=torch.bfloat16, device="cuda")
        plan = moin.Plan(ctx)

        def call(out):
            plan.build(inp.seq_offsets, eids, inp.wl.T, inp.wl.E)
            moin.moin_lora_linear_planned(ctx, plan, x, inp.W, inp.A_stack, inp.B_stack, 2.0, out=out)

        assert ctx.workspace_bytes() == 0
        torch.cuda.synchronize()
        print("[gpu] graph growth: capture on an empty context is refused", flush=True)
        graph = torch.cuda.CUDAGraph()
        refused = []
        with torch.cuda.graph(graph):
            for step in (lambda: plan.build(inp.seq_offsets, eids, inp.wl.T, inp.wl.E),):
                try:
                    step()
                except moin.MoinError as e:
                    refused.append(e.code)
        assert refused == [-6], refused
        assert ctx.workspace_bytes() == 0
        del graph
        # reserve outside the capture: the plan for up to 128 sequences, the workspace from an eager call
        plan.reserve(128, 128, inp.wl.E)
        y_eager = torch.empty_like(y_graph)
        call(y_eager)
        ctx.check()
        need = ctx.workspace_bytes()
        assert need > 0
        ctx.reserve_workspace(need)            # no-op: already that large
        assert ctx.workspace_bytes() == need
        print("[gpu] graph growth: capture after reserving", flush=True)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call(y_graph)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y_graph.view(torch.int16), y_eager.view(torch.int16))
        # a larger eager batch on the same context and plan: both buffers are replaced ...
        print("[gpu] graph growth: larger eager call, then replay", flush=True)
        plan_b = plan.build(big.seq_offsets, big.expert_ids, big.wl.T, big.wl.E)
        yb = moin.moin_lora_linear_planned(ctx, plan_b, big.x, big.W, big.A_stack, big.B_stack, 2.0)
        ctx.check()
        assert ctx.workspace_bytes() > need
        gc.compare_linear(yb, gc.oracle_rows(big), what="graph_grow/big eager")
        # ... and the graph still replays on the blocks it recorded, with new inputs in place
        x.copy_(torch.randn(x.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(9))
                .to(torch.bfloat16))
        eids.copy_(inp.expert_ids.flip(0))
        y_graph.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        ref = gc.oracle_rows(wl.LinearInputs(inp.wl, x, inp.W, inp.A_stack, inp.B_stack, inp.seq_offsets, eids))
        gc.compare_linear(y_graph, ref, what="graph_grow/replay after growth")
        plan.close()
    finally:
        ctx.close()


def _captured_on_a_fresh_context(what, prepare, call, outs):
    """call(ctx, state) is recorded on a context that has made no call yet, and replayed on changed inputs."""
    ctx, eager = moin.Context(0), gc.ctx()
    try:
        st, ref = prepare(ctx), prepare(eager)
        torch.cuda.synchronize()
        print(f"[gpu] graph {what}: capture on a fresh context", flush=True)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call(ctx, st)
        for rep in range(3):
            print(f"[gpu] graph {what}: replay {rep}", flush=True)
            g = torch.Generator(device="cuda").manual_seed(20 + rep)
            st["emb"].copy_(torch.randn(st["emb"].shape, device="cuda", generator=g))
            ref["emb"].copy_(st["emb"])
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            call(eager, ref)
            ctx.check()
            eager.check()
            for a, b in zip(outs(st), outs(ref)):
                assert torch.equal(a, b), f"{what}: replay {rep}"
    finally:
        torch.cuda.synchronize()
        ctx.close()


def _fp32_routing(ctx, N=48, K=300, D=96):
    r = wl.make_route_inputs(wl.RouteWorkload("graph_f32", N, K, D, "f32", False, 91), "cuda")
    i32 = lambda n: torch.empty(n, dtype=torch.int32, device="cuda")
    return dict(emb=r.emb.clone(), cent=r.centroids.clone(), out=(i32(N), i32(N), i32(K)))


def test_small_fp32_routing_call_needs_no_call_before_its_capture():
    _captured_on_a_fresh_context(
        "f32 route", _fp32_routing, lambda c, s: moin.moin_route(c, s["emb"], s["cent"], out=s["out"]),
        lambda s: s["out"])


def test_small_fp32_route_and_plan_call_needs_the_plan_reserved_only():
    S, T, E = 48, 96, 300
    off = torch.arange(0, T + 1, 2, dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(92)
    W = torch.randn((64, 64), device="cuda", generator=g).to(torch.bfloat16)
    A = torch.randn((E, 16, 64), device="cuda", generator=g).to(torch.bfloat16)
    B = torch.randn((E, 64, 16), device="cuda", generator=g).to(torch.bfloat16)
    x = torch.randn((T, 64), device="cuda", generator=g).to(torch.bfloat16)

    def prepare(ctx):
        st = _fp32_routing(ctx, N=S, K=E)
        st["plan"], st["y"] = moin.Plan(ctx), torch.empty((T, 64), dtype=torch.bfloat16, device="cuda")
        st["plan"].reserve(S, T, E)
        ctx.reserve_workspace(1 << 20)
        return st

    def call(ctx, st):
        moin.moin_route_plan(ctx, st["plan"], st["emb"], st["cent"], off, T, E, out=st["out"])
        moin.moin_lora_linear_planned(ctx, st["plan"], x, W, A, B, 2.0, out=st["y"])

    _captured_on_a_fresh_context("f32 route + plan", prepare, call, lambda s: (*s["out"], s["y"].view(torch.int16)))


def test_kmeans_on_few_fp32_points_needs_the_workspace_reserved_only():
    N, K, D = 900, 40, 64

    def prepare(ctx):
        st = _fp32_routing(ctx, N=N, K=K, D=D)
        st["first"] = st["cent"].clone()
        ctx.reserve_workspace(1 << 22)
        return st

    def call(ctx, st):
        st["cent"].copy_(st["first"])
        st["got"] = moin.moin_kmeans_fit(ctx, st["emb"], st["cent"], 2)

    _captured_on_a_fresh_context("f32 kmeans", prepare, call, lambda s: (*s["got"], s["cent"]))
