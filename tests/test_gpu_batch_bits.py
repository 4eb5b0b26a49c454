"""A sequence's results are the same bits among a few others and at the head of larger batches, whichever kernels each size
takes: adapters in full, every width of the shrink, own ranks, projections that share their input, and a quantised
base whose codes are made on the way or given."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu

FEW = [300, 256, 31, 511, 130]
BATCHES = [FEW, FEW + [400] * 20, FEW + [400] * 140]
MANY = BATCHES[-1]
E = 5


def _inputs(d_in, d_out, r, seed):
    ids = np.array([2, 0, 1, 3, -1] + [0, 1, 2, 3, -1] * 28, dtype=np.int32)
    w = wl.LinearWorkload("bits", d_in, d_out, r, E, MANY, "uniform", scale=2.0, seed=seed)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    inp.A_stack[4] = float("nan")   # (no sequence uses it)
    inp.B_stack[4] = float("nan")
    return inp


def _plans(inp, ranks):
    rk = None if ranks is None else torch.tensor(ranks, dtype=torch.int32, device="cuda")
    return [moin.Plan(gc.ctx()).build(inp.seq_offsets[:len(b) + 1].contiguous(), inp.expert_ids[:len(b)].contiguous(),
                                      sum(b), E, rank_of_expert=rk) for b in BATCHES]


@pytest.mark.parametrize("d_in,r,ranked", [(64, 8, False), (192, 24, True), (704, 40, False), (2048, 16, False),
                                           (2048, 64, True), (1344, 72, True), (2048, 128, False)])
def test_bf16_base(d_in, r, ranked):
    inps = [_inputs(d_in, d_out, r, 7 + d_out) for d_out in (72, 136)]
    x = inps[0].x
    plans = _plans(inps[0], [r, 8, max(8, r - 8), 8 * (r // 16), r] if ranked else None)
    print(f"[gpu] bits by batch, bf16 base, d_in={d_in} r={r} ranked={ranked}", flush=True)

    def calls(plan, x):
        one = moin.moin_lora_linear_planned(gc.ctx(), plan, x, inps[0].W, inps[0].A_stack, inps[0].B_stack, 2.0,
                                            y_dtype=torch.float32)
        two = moin.moin_lora_linear_planned_shared(gc.ctx(), plan, x, [i.W for i in inps], [i.A_stack for i in inps],
                                                   [i.B_stack for i in inps], 2.0, y_dtype=torch.float32)
        return [one, *two]

    got = [calls(plan, x[:sum(b)].contiguous()) for plan, b in zip(plans, BATCHES)]
    gc.ctx().check()
    for ys, b in zip(got, BATCHES):
        assert torch.equal(ys[0], ys[1])
        for y, whole in zip(ys, got[-1]):
            assert bool(torch.isfinite(whole).all()) and torch.equal(y, whole[:sum(b)])
    for plan in plans:
        plan.close()


@pytest.mark.parametrize("d_in,r,ranks", [(256, 64, [64, 8, 40, 0, 64]), (1408, 128, [128, 72, 64, 8, 128]), (2048, 64, None)])
def test_quantised_base(d_in, r, ranks):
    inp = _inputs(d_in, 136, r, 3)
    Wq, Ws = moin.moin_mx_quantize(gc.ctx(), inp.W, blocked=True)
    plans = _plans(inp, ranks)
    print(f"[gpu] bits by batch, quantised base, d_in={d_in} r={r} ranks={ranks}", flush=True)

    def calls(plan, x):
        xq = torch.zeros((x.shape[0], d_in), dtype=torch.uint8, device="cuda")
        xs = torch.zeros((d_in // 128, x.shape[0], 4), dtype=torch.uint8, device="cuda")
        call = lambda **kw: moin.moin_lora_linear_mx_planned(gc.ctx(), plan, x, Wq, Ws, inp.A_stack, inp.B_stack, 2.0,
                                                             y_dtype=torch.float32, **kw)
        made, given = call(xq=xq, xs=xs, emit=True), call(xq=xq, xs=xs)
        q, s = moin.moin_mx_quantize(gc.ctx(), x, blocked=True)
        assert torch.equal(made, given) and torch.equal(xq, q.view(torch.uint8)) and torch.equal(xs, s)
        return made

    got = [calls(plan, inp.x[:sum(b)].contiguous()) for plan, b in zip(plans, BATCHES)]
    gc.ctx().check()
    assert bool(torch.isfinite(got[-1]).all())
    for y, b in zip(got, BATCHES):
        assert torch.equal(y, got[-1][:sum(b)])
    for plan in plans:
        plan.close()
