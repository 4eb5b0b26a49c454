"""The prefill kernel on 128 x 128 tiles: row counts around a tile and a plan tile, widths and contraction lengths on
both sides of a block, ranks that end inside one, with one tile per compute unit and with more, on prefill and on plain
row tiles; against torch in fp64.  And its bits against the larger tiles'."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc
from tests.test_gpu_decode_stream import _check, _reference

pytestmark = pytest.mark.gpu

LENS = [300, 256, 1, 130, 511, 128, 129, 255, 127, 640]
IDS = np.array([2, 0, -1, 2, 3, 1, 1, 0, 3, 2], dtype=np.int32)
E = 5


def _run(lens, ids, d_in, d_out, r, ranked, f32):
    w = wl.LinearWorkload("mid", d_in, d_out, r, E, lens, "uniform", scale=2.0, seed=d_in + d_out + r)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    rk = torch.tensor([r, 8, max(8, r - 8), 0, 8], dtype=torch.int32, device="cuda") if ranked else None
    inp.A_stack[4] = float("nan")   # (no sequence uses it)
    inp.B_stack[4] = float("nan")
    print(f"[gpu] prefill on 128 x 128 tiles {len(lens)} x {d_in}->{d_out} r={r} ranked={ranked} f32={f32}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32 if f32 else torch.bfloat16, rank_of_expert=rk)
    gc.ctx().check()
    return y, _reference(inp, ids, lens, rk, r)


@pytest.mark.parametrize("d_in,d_out,r,ranked,f32", [
    (8, 8, 8, False, True), (56, 136, 24, True, True), (64, 128, 64, False, True), (72, 120, 72, False, False),
    (200, 264, 40, True, True), (256, 1416, 16, False, True), (1000, 2048, 32, True, True), (2048, 256, 128, False, False),
    (2048, 2000, 64, True, True), (1416, 1000, 136, False, True)])
def test_edges(d_in, d_out, r, ranked, f32):
    y, ref = _run(LENS, IDS, d_in, d_out, r, ranked, f32)
    if f32:
        _check(y, ref, d_in, r)
    else:   # rounded to bf16: half a unit of the last of 8 bits
        assert bool(((y.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all())


@pytest.mark.parametrize("lens,d_out", [([129, 200, 20, 256, 300] * 15, 200), ([140, 128, 250] * 60, 72), ([20, 400] * 125, 8)])
def test_many_plan_tiles(lens, d_out):   # 90, 180, and more than the 256 whose empty halves are left out
    ids = (np.arange(len(lens)) % E - 1).astype(np.int32)
    y, ref = _run(lens, ids, 72, d_out, 24, True, True)
    _check(y, ref, 72, 24)


@pytest.mark.parametrize("S,d_in,d_out", [(1025, 1000, 136), (1300, 2048, 264), (3000, 72, 1000)])
def test_plain_tiles(S, d_in, d_out):
    ids = (np.arange(S) % E - 1).astype(np.int32)   # -1 .. 3
    y, ref = _run([1] * S, ids, d_in, d_out, 16, False, True)
    _check(y, ref, d_in, 16)


@pytest.mark.parametrize("S,d_in,d_out,r,kernel", [
    (1300, 5640, 256, 32, moin.K_DECODE_BASE),   # long ragged rows, few tiles: the contraction in parts
    (1300, 5640, 256, 0, moin.K_LINEAR), (1300, 5640, 2048, 32, moin.K_LINEAR), (1300, 1000, 256, 32, moin.K_LINEAR), (1300, 5632, 256, 32, moin.K_LINEAR)])
def test_base_product_of_gathered_batches(S, d_in, d_out, r, kernel):
    ids, ctx = (np.arange(S) % E - 1 if r else np.full(S, -1)).astype(np.int32), gc.ctx()
    w = wl.LinearWorkload("mid", d_in, d_out, max(r, 8), E, [1] * S, "uniform", scale=2.0, seed=d_in + r)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    A, B = (inp.A_stack, inp.B_stack) if r else (None, None)
    print(f"[gpu] base product of {S} tokens {d_in}->{d_out} r={r}", flush=True)
    ctx.timing_reset()
    ctx.timing_enable(True)
    try:
        y = moin.moin_lora_linear(ctx, inp.x, inp.seq_offsets, inp.expert_ids, inp.W, A, B, 2.0, y_dtype=torch.float32)
        ctx.check()
        launches = {k: ctx.timing_read(k)[1] for k in (moin.K_DECODE_BASE, moin.K_LINEAR)}
    finally:
        ctx.timing_enable(False)
    assert launches == {moin.K_DECODE_BASE: int(kernel == moin.K_DECODE_BASE), moin.K_LINEAR: int(kernel == moin.K_LINEAR)}
    _check(y, _reference(inp, ids, [1] * S, None, r), d_in, max(r, 8))


@pytest.mark.parametrize("r", [64, 24])
def test_same_bits_as_the_larger_tiles(r):
    d_in, d_out = 192, 4096
    ids = np.array([0, 1, 2, 3] * 8, dtype=np.int32)
    w = wl.LinearWorkload("mid", d_in, d_out, r, E, [400] * 32, "uniform", scale=2.0, seed=r)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)   # 4096 tiles
    call = lambda x, off, e: moin.moin_lora_linear(gc.ctx(), x, off, e, inp.W, inp.A_stack, inp.B_stack, 2.0,
                                                   y_dtype=torch.float32)
    print(f"[gpu] 128 x 128 and 256 x 256 tiles, r={r}", flush=True)
    y = call(inp.x, inp.seq_offsets, inp.expert_ids)
    # 384 tiles
    few = call(inp.x[:1200].contiguous(), inp.seq_offsets[:4].contiguous(), inp.expert_ids[:3].contiguous())
    gc.ctx().check()
    assert torch.equal(few, y[:1200])
