"""Stacks whose rank is not a multiple of 64 on 128 x 128 tiles (on the larger ones: test_gpu_large_batches.py): one block and several, the first and
the last rank of a block, experts of smaller rank (other experts and rows past the own rank filled with NaN where they
are never read), ragged tiles, several projections in one call; against torch in fp64."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc
from tests.test_gpu_decode_stream import _check, _reference

pytestmark = pytest.mark.gpu

LENS = [300, 256, 1, 130, 511]
IDS = np.array([2, 0, -1, 2, 3], dtype=np.int32)
E = 5


def _inputs(d_in, d_out, r, seed):
    w = wl.LinearWorkload("ragged", d_in, d_out, r, E, LENS, "uniform", scale=2.0, seed=seed)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=IDS)
    for e in (1, 4):   # no sequence uses these
        inp.A_stack[e] = float("nan")
        inp.B_stack[e] = float("nan")
    return inp


@pytest.mark.parametrize("d_in,d_out,r,ranked,f32", [
    (128, 256, 8, False, True), (256, 264, 16, False, True), (256, 264, 40, True, True), (192, 520, 56, False, False),
    (256, 72, 72, True, True), (128, 256, 120, False, True), (256, 264, 136, True, True), (2048, 512, 200, False, True)])
def test_rank_not_a_multiple_of_64(d_in, d_out, r, ranked, f32):
    inp = _inputs(d_in, d_out, r, d_in + r)
    rk = torch.tensor([8, 8, max(8, r - 8), 0, 8], dtype=torch.int32, device="cuda") if ranked else None
    if ranked:
        inp.A_stack[2, r - 8:] = float("nan") if r > 8 else 0.0
    print(f"[gpu] prefill {d_in}->{d_out} r={r} ranked={ranked}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32 if f32 else torch.bfloat16, rank_of_expert=rk)
    gc.ctx().check()
    ref = _reference(inp, IDS, LENS, rk, r)
    if f32:
        _check(y, ref, d_in, r)
    else:   # rounded to bf16: half a unit of the last of 8 bits
        assert bool(((y.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all())


def test_shared_call():
    d_in, r, widths = 256, 24, (264, 520, 16)
    ins = [_inputs(d_in, d, r, 90 + d) for d in widths]
    for i in ins[1:]:
        i.x.copy_(ins[0].x)
    T = sum(LENS)
    plan = moin.Plan(gc.ctx())
    plan.build(ins[0].seq_offsets, ins[0].expert_ids, T, E)
    print("[gpu] prefill shared, r=24", flush=True)
    ys = moin.moin_lora_linear_planned_shared(gc.ctx(), plan, ins[0].x, [i.W for i in ins], [i.A_stack for i in ins],
                                              [i.B_stack for i in ins], 2.0, y_dtype=torch.float32)
    gc.ctx().check()
    for y, i in zip(ys, ins):
        _check(y, _reference(i, IDS, LENS, None, r), d_in, r)
