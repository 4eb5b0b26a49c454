"""Batches that are grouped both ways, in row tiles and by expert: calls on both sides of each line between the two, by
tokens, tokens per sequence, rank and contraction length; single calls, calls that share their input (the same bits) and
an MXFP8 base; own ranks, base-only sequences and sequences of uneven length; against torch in fp64."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc
from tests.test_gpu_decode_stream import _check, _reference

pytestmark = pytest.mark.gpu
E = 6


def _batch(lens, d_in, d_out, r, ranked):
    ids = (np.arange(len(lens)) % (E - 1) - 1).astype(np.int32)   # -1 .. 3: adapters 4 and 5 have no sequence
    w = wl.LinearWorkload("both", d_in, d_out, r, E, lens, "uniform", scale=2.0, seed=d_in + r + sum(lens))
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    inp.A_stack[4] = float("nan")
    inp.B_stack[5] = float("inf")
    rk = torch.tensor([r, 8, max(8, r - 8), 0, 8, 8], dtype=torch.int32, device="cuda") if ranked else None
    return inp, ids, rk


def _counted(ctx, call):
    """The call's result, and whether it took row tiles."""
    ctx.timing_reset()
    ctx.timing_enable(True)
    try:
        y = call()
        ctx.check()
        tiles, gathered = (ctx.timing_read(k)[1] for k in (moin.K_SHRINK, moin.K_DECODE_SHRINK))
    finally:
        ctx.timing_enable(False)
    assert (tiles > 0) != (gathered > 0)
    return y, tiles > 0


@pytest.mark.parametrize("lens,d_in,r,tiles", [
    ([319], 64, 128, False), ([320], 64, 128, True), ([64] * 5, 1000, 64, True), ([64] * 5 + [63], 1024, 64, False),
    ([383], 1024, 8, False), ([384], 1024, 8, True), ([20, 140] * 5, 72, 40, True), ([19, 140] * 5, 72, 40, False),
    ([300, 19], 2048, 128, False), ([300, 20], 2048, 128, True), ([76] * 5, 1032, 64, False), ([77] * 5, 1032, 64, True),
    ([10, 134] * 7, 2048, 72, True), ([9, 134] * 7, 2048, 72, False), ([96] * 8, 2048, 16, True), ([95, 96] * 4, 2048, 16, False), ([153] * 5, 2048, 32, False), ([154] * 5, 2048, 32, True),
    ([639], 5632, 128, False), ([640], 5632, 128, True), ([1024], 5632, 16, False), ([1025], 5632, 16, True),
    ([80] * 13, 2048, 48, True), ([79] * 13, 2048, 48, False), ([127] * 33, 1032, 40, False), ([127] * 33, 1032, 48, True),
    ([400] * 2, 2048, 136, False), ([1, 500, 0, 3, 150], 2048, 128, True)])
def test_both_sides_of_each_line(lens, d_in, r, tiles):
    ranked = len(lens) % 2 == 0
    inp, ids, rk = _batch(lens, d_in, 136, r, ranked)
    W2, A2, B2 = inp.W[:72].contiguous(), inp.A_stack, inp.B_stack[:, :72].contiguous()
    print(f"[gpu] both groupings T={sum(lens)} S={len(lens)} {d_in}->136 r={r}", flush=True)
    ctx = gc.ctx()
    plan = moin.Plan(ctx).build(inp.seq_offsets, inp.expert_ids, sum(lens), E, rank_of_expert=rk)
    y, took = _counted(ctx, lambda: moin.moin_lora_linear_planned(ctx, plan, inp.x, inp.W, inp.A_stack, inp.B_stack, 2.0,
                                                                  y_dtype=torch.float32))
    assert took == tiles
    _check(y, _reference(inp, ids, lens, rk, r), d_in, r)
    two = moin.moin_lora_linear_planned_shared(ctx, plan, inp.x, [inp.W, W2], [inp.A_stack, A2], [inp.B_stack, B2], 2.0,
                                               y_dtype=torch.float32)
    one = moin.moin_lora_linear_planned(ctx, plan, inp.x, W2, A2, B2, 2.0, y_dtype=torch.float32)
    base = moin.moin_lora_linear_planned(ctx, plan, inp.x, inp.W, None, None, 2.0, y_dtype=torch.float32)
    ctx.check()
    assert torch.equal(two[0], y) and torch.equal(two[1], one)
    _check(two[1], y[:, :72].double(), d_in, r)
    _check(base, inp.x.double() @ inp.W.double().T, d_in, r)
    plan.close()


@pytest.mark.parametrize("lens,r,tiles", [([64] * 7, 64, False), ([72] * 8, 64, True), ([5, 315], 128, True), ([5, 314], 128, False)])
def test_quantised_base(lens, r, tiles):
    d_in, T, ctx = 1152, sum(lens), gc.ctx()
    inp, ids, _ = _batch(lens, d_in, 200, r, False)
    Wq, Ws = moin.moin_mx_quantize(ctx, inp.W, blocked=True)
    plan = moin.Plan(ctx).build(inp.seq_offsets, inp.expert_ids, T, E)
    xq, xs = (torch.zeros(s, dtype=torch.uint8, device="cuda") for s in ((T, d_in), (d_in // 128, T, 4)))
    print(f"[gpu] both groupings, quantised base, T={T} S={len(lens)} r={r}", flush=True)
    call = lambda **kw: moin.moin_lora_linear_mx_planned(ctx, plan, inp.x, Wq, Ws, inp.A_stack, inp.B_stack, 2.0,
                                                         y_dtype=torch.float32, **kw)
    made, took = _counted(ctx, lambda: call(xq=xq, xs=xs, emit=True))
    assert took == tiles
    q, s = moin.moin_mx_quantize(ctx, inp.x, blocked=True)
    assert torch.equal(xq, q) and torch.equal(xs, s)
    assert torch.equal(call(xq=xq, xs=xs), made) and torch.equal(call(), made)

    def values(codes, scales):   # E4M3 codes times 2^(scale - 127), the scale bytes of a row's 128 values side by side
        e = scales.permute(1, 0, 2).reshape(codes.shape[0], -1).repeat_interleave(32, dim=1)
        return codes.view(torch.float8_e4m3fn).double() * torch.exp2(e.double() - 127)

    on_x = _reference(inp, ids, lens, None, r) - inp.x.double() @ inp.W.double().T   # the adapters' share
    _check(made, on_x + values(xq, xs) @ values(Wq, Ws).T, d_in, r)
    plan.close()


@pytest.mark.parametrize("first,then,r", [([500], [300], 128), ([130], [128], 16), ([96] * 10, [80] * 10, 64)])
@pytest.mark.parametrize("kind", ["plain", "shared", "mx"])
def test_the_largest_batch_sizes_the_workspace_for_smaller_ones(first, then, r, kind):
    if kind == "mx" and r % 64:
        pytest.skip("not a rank of the quantised base")
    ctx = moin.Context(0)
    try:
        sizes = []
        for lens in (first, then):
            inp, _, _ = _batch(lens, 2048, 2048, r, False)
            plan = moin.Plan(ctx).build(inp.seq_offsets, inp.expert_ids, sum(lens), E)
            if kind == "mx":
                Wq, Ws = moin.moin_mx_quantize(ctx, inp.W, blocked=True)
                moin.moin_lora_linear_mx_planned(ctx, plan, inp.x, Wq, Ws, inp.A_stack, inp.B_stack, 2.0)
            elif kind == "shared":
                moin.moin_lora_linear_planned_shared(ctx, plan, inp.x, [inp.W] * 2, [inp.A_stack] * 2, [inp.B_stack] * 2, 2.0)
            else:
                moin.moin_lora_linear_planned(ctx, plan, inp.x, inp.W, inp.A_stack, inp.B_stack, 2.0)
            ctx.check()
            sizes.append(ctx.workspace_bytes())
            plan.close()
        assert sizes[1] == sizes[0]
    finally:
        torch.cuda.synchronize()
        ctx.close()
