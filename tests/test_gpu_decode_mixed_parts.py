"""Calls of up to 128 tokens whose projections' base products are cut into different numbers of parts: two launches, the bits of
single calls; widths on both sides of the rule for few tokens, ranks in every form of the expand, own ranks, base-only
sequences; against torch in fp64."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests.test_gpu_decode_stream import _check, _reference

pytestmark = pytest.mark.gpu
E = 6


@pytest.mark.parametrize("T,d_in,d_outs,r,ranked", [
    (33, 2048, (8200, 264), 16, False), (88, 2048, (8192, 1024, 1024), 64, True), (89, 2048, (8192, 1024, 1024), 128, False),
    (80, 2048, (2048, 8208), 40, True), (128, 2048, (72, 8200, 2048, 8), 128, True), (128, 1024, (8208, 264), 136, False),
    (64, 1088, (264, 8264), 24, False), (100, 2112, (8264, 16), 200, True), (128, 512, (264, 8456), 32, False),
    (129, 2048, (8192, 1024), 64, False), (20, 4224, (22016, 264), 32, True)])
def test_projections_of_different_parts_share_their_launches(T, d_in, d_outs, r, ranked):
    lens = [T // 3, 1, T - T // 3 - 12, 4, 7]
    ids = np.array([1, -1, 3, 0, 1], dtype=np.int32)
    inps = [wl.make_linear_inputs(wl.LinearWorkload("mixed", d_in, d, r, E, lens, "uniform", scale=2.0, seed=d + T), "cuda", expert_ids=ids)
            for d in d_outs]
    x = inps[0].x
    for i in inps:
        i.x = x
        i.A_stack[4], i.B_stack[5] = float("nan"), float("inf")   # (no sequence uses them)
    rk = torch.tensor([r, 8, 0, max(8, r - 8), 8, 8], dtype=torch.int32, device="cuda") if ranked else None
    print(f"[gpu] mixed parts T={T} {d_in}->{d_outs} r={r} ranked={ranked}", flush=True)
    ctx = moin.Context(0)
    try:
        plan = moin.Plan(ctx).build(inps[0].seq_offsets, inps[0].expert_ids, T, E, rank_of_expert=rk)
        for dt in (torch.float32, torch.bfloat16):
            ctx.timing_enable(True)
            ctx.timing_reset()
            ys = moin.moin_lora_linear_planned_shared(ctx, plan, x, [i.W for i in inps], [i.A_stack for i in inps],
                                                      [i.B_stack for i in inps], 2.0, y_dtype=dt)
            ctx.check()
            assert [ctx.timing_read(k)[1] for k in (moin.K_DECODE_SHRINK, moin.K_DECODE_EXPAND)] == [1, 1]
            ctx.timing_enable(False)
            for y, i in zip(ys, inps):
                one = moin.moin_lora_linear_planned(ctx, plan, x, i.W, i.A_stack, i.B_stack, 2.0, y_dtype=dt)
                assert torch.equal(y, one)
                if dt == torch.float32:
                    _check(y, _reference(i, ids, lens, rk, r), d_in, r)
            ctx.check()
        plan.close()
    finally:
        torch.cuda.synchronize()
        ctx.close()
