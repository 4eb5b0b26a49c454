"""The shrink of few row tiles, a wave per 32 tokens and 16 columns by itself or (in the batches of 30 and 40 sequences) in tiles of
64 x 32 and 64 x 64, on a quantised base 32 x 64 and 64 x 64: row counts around a
tile, fewer blocks of 64 than stages to many more, every width, ranks that end inside one, on a bf16 and (codes made on the
way, and given) an MXFP8 base; against torch in fp64, and codes against the quantiser's."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc
from tests.test_gpu_decode_stream import _check, _reference

pytestmark = pytest.mark.gpu

LENS = [300, 256, 1, 31, 511, 32, 33, 255, 129, 640]
IDS = np.array([2, 0, -1, 2, 3, 1, 1, -1, 3, 2], dtype=np.int32)
E = 5


def _inputs(d_in, d_out, r, times=1):
    w = wl.LinearWorkload("split", d_in, d_out, r, E, LENS * times, "uniform", scale=2.0, seed=d_in + r)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=np.tile(IDS, times))
    inp.A_stack[4] = float("nan")   # (no sequence uses it)
    inp.B_stack[4] = float("nan")
    return inp


@pytest.mark.parametrize("d_in,r,ranked", [(64, 8, False), (128, 16, True), (192, 32, False), (320, 40, True), (704, 64, False),
                                           (2048, 64, True), (256, 72, True), (1344, 96, False), (5632, 128, True), (512, 16, False),
                                           (576, 40, True)])
def test_against_fp64(d_in, r, ranked):
    inp = _inputs(d_in, 72, r)
    rk = torch.tensor([r, 8, max(8, r - 8), 0, 8], dtype=torch.int32, device="cuda") if ranked else None
    print(f"[gpu] split shrink d_in={d_in} r={r} ranked={ranked}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32, rank_of_expert=rk)
    gc.ctx().check()
    _check(y, _reference(inp, IDS, LENS, rk, r), d_in, r)


@pytest.mark.parametrize("d_in,r,ranked,times", [
    (64, 24, False, 4), (192, 32, True, 4), (256, 40, False, 3), (320, 64, True, 3), (1408, 48, True, 3),
    (128, 40, True, 4), (256, 64, False, 4), (704, 72, False, 4), (2048, 64, False, 4), (1344, 128, True, 4), (192, 96, True, 4)])
def test_wider_patches_against_fp64(d_in, r, ranked, times):
    inp, ids, lens = _inputs(d_in, 72, r, times), np.tile(IDS, times), LENS * times
    rk = torch.tensor([r, 8, max(8, r - 8), 0, 8], dtype=torch.int32, device="cuda") if ranked else None
    print(f"[gpu] shrink, tiles of several waves, d_in={d_in} r={r} ranked={ranked}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32, rank_of_expert=rk)
    gc.ctx().check()
    _check(y, _reference(inp, ids, lens, rk, r), d_in, r)


@pytest.mark.parametrize("d_in,r,times", [(256, 64, 1), (384, 128, 1), (2048, 64, 1), (5632, 128, 1), (256, 64, 4), (896, 128, 4)])
def test_quantised_base(d_in, r, times):
    inp, ctx, T = _inputs(d_in, 72, r, times), gc.ctx(), sum(LENS) * times
    Wq, Ws = moin.moin_mx_quantize(ctx, inp.W, blocked=True)
    want_q, want_s = moin.moin_mx_quantize(ctx, inp.x, blocked=True)
    plan = moin.Plan(ctx).build(inp.seq_offsets, inp.expert_ids, T, E)
    xq = torch.zeros((T, d_in), dtype=torch.uint8, device="cuda")
    xs = torch.zeros((d_in // 128, T, 4), dtype=torch.uint8, device="cuda")
    call = lambda **kw: moin.moin_lora_linear_mx_planned(ctx, plan, inp.x, Wq, Ws, inp.A_stack, inp.B_stack, 2.0,
                                                         y_dtype=torch.float32, **kw)
    print(f"[gpu] split shrink with codes d_in={d_in} r={r} times={times}", flush=True)
    y0, y1 = call(xq=xq, xs=xs, emit=True), call(xq=xq, xs=xs)
    ctx.check()
    assert torch.equal(xq, want_q.view(torch.uint8)) and torch.equal(xs, want_s) and torch.equal(y0, y1)
    # the adapter term, from the same call without adapters (its products of codes are the same sums)
    none = torch.full_like(inp.expert_ids, -1)
    base = moin.moin_lora_linear_mx(ctx, inp.x, inp.seq_offsets, none, Wq, Ws, inp.A_stack, inp.B_stack, 2.0,
                                    y_dtype=torch.float32)
    ctx.check()
    zero_w = wl.LinearInputs(inp.wl, inp.x, torch.zeros_like(inp.W), inp.A_stack, inp.B_stack, inp.seq_offsets,
                             inp.expert_ids)
    term = _reference(zero_w, np.tile(IDS, times), LENS * times, None, r)
    ref = base.double() + term
    # u as a bf16 pair (2^-17) and fp32 sums of d_in + r products, against the largest output, taken four times
    bound = 4 * (d_in ** 0.5 + 128) * 2.0 ** -24
    assert float((y0.double() - ref).abs().max()) <= bound * float(ref.abs().max())
    plan.close()
