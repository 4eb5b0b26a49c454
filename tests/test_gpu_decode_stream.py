"""The streaming decode kernels where they change: base product as slabs or tiles (16 / 17 and 32 / 33 tokens, widths on
both sides of the rule), rows of one, two and a ragged number of steps, every width of the expand, records of several
token blocks, ranks below the stacks' and sequences without an adapter; against torch in fp64."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


def _batch(lens, E, seed, hot=0.3):
    rng = np.random.default_rng(seed)
    ids = rng.integers(-1, E, size=len(lens)).astype(np.int32)
    ids[rng.random(len(lens)) < hot] = E - 1
    ranks = lambda r: torch.from_numpy((8 * rng.integers(0, r // 8 + 1, size=E)).astype(np.int32)).cuda()
    return ids, ranks


def _reference(inp, ids, lens, ranks, r):
    tok = torch.from_numpy(np.repeat(ids, lens).astype(np.int64)).cuda()
    x = inp.x.double()
    ref = x @ inp.W.double().T
    for e in sorted(set(ids.tolist()) - {-1}):
        at = (tok == e).nonzero()[:, 0]
        k = r if ranks is None else int(ranks[e])
        u = x[at] @ inp.A_stack[e, :k].double().T
        ref[at] += 2.0 * u @ inp.B_stack[e, :, :k].double().T
    return ref


def _check(y, ref, d_in, r):
    # fp32 sums of d_in + r products and u as a bf16 pair (2^-17): both stay under (sqrt(d_in) + 2^7) * 2^-24 of the
    # largest output, taken four times
    bound = 4 * (d_in ** 0.5 + 128) * 2.0 ** -24
    assert float((y.double() - ref).abs().max()) <= bound * float(ref.abs().max())


@pytest.mark.parametrize("T,d_in,d_out,r,ranked", [
    (1, 2048, 256, 128, False), (16, 2048, 72, 40, True), (17, 2048, 4096, 64, False), (17, 2048, 4104, 64, True),
    (32, 72, 200, 8, False), (33, 72, 200, 24, True), (32, 2112, 264, 72, True), (5, 5632, 136, 128, True),
    (12, 4104, 88, 136, False), (100, 5632, 136, 32, False), (300, 1000, 328, 128, True), (1024, 256, 40, 96, True)])
def test_small_batches(T, d_in, d_out, r, ranked):
    lens = [1] * T
    E = 9
    ids, ranks = _batch(lens, E, T + d_in)
    w = wl.LinearWorkload("stream", d_in, d_out, r, E, lens, "uniform", scale=2.0, seed=T + r)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    rk = ranks(r) if ranked else None
    print(f"[gpu] decode stream T={T} {d_in}->{d_out} r={r} ranked={ranked}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32, rank_of_expert=rk)
    gc.ctx().check()
    _check(y, _reference(inp, ids, lens, rk, r), d_in, r)


@pytest.mark.parametrize("S,E,d_in,r,ranked", [(1100, 600, 2048, 128, True), (1300, 700, 2112, 40, False),
                                               (5000, 2500, 256, 64, True)])
def test_large_batches_with_records_of_several_blocks(S, E, d_in, r, ranked):
    lens = [1] * S
    ids, ranks = _batch(lens, E, S, hot=0.1)
    w = wl.LinearWorkload("stream", d_in, 200, r, E, lens, "uniform", scale=2.0, seed=S)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    rk = ranks(r) if ranked else None
    print(f"[gpu] decode stream S={S} E={E} d_in={d_in} r={r}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32, rank_of_expert=rk)
    gc.ctx().check()
    _check(y, _reference(inp, ids, lens, rk, r), d_in, r)


@pytest.mark.parametrize("T", [20, 40])
def test_shared_call_of_widths_on_both_sides_of_the_slab_rule(T):
    lens, E, d_in, r = [1] * T, 6, 256, 32
    ids, _ = _batch(lens, E, T)
    ins = [wl.make_linear_inputs(wl.LinearWorkload("stream", d_in, d, r, E, lens, "uniform", scale=2.0, seed=50 + d),
                                 "cuda", expert_ids=ids) for d in (264, 4112, 48)]
    for i in ins[1:]:
        i.x.copy_(ins[0].x)
    plan = moin.Plan(gc.ctx())
    plan.build(ins[0].seq_offsets, ins[0].expert_ids, T, E)
    print(f"[gpu] decode stream shared T={T}", flush=True)
    ys = moin.moin_lora_linear_planned_shared(gc.ctx(), plan, ins[0].x, [i.W for i in ins], [i.A_stack for i in ins],
                                              [i.B_stack for i in ins], 2.0, y_dtype=torch.float32)
    gc.ctx().check()
    for y, i in zip(ys, ins):
        _check(y, _reference(i, ids, lens, None, r), d_in, r)


@pytest.mark.parametrize("d_in,r", [(256, 32), (2048, 64), (2048, 136)])
def test_a_shared_call_with_slabs_and_tiles_takes_two_launches(d_in, r):
    # 17 tokens: 4096 outputs and fewer come from slabs of W, more from tiles (at 2048 inputs in two parts)
    T, E = 17, 6
    lens = [1] * T
    ids, _ = _batch(lens, E, T)
    ins = [wl.make_linear_inputs(wl.LinearWorkload("stream", d_in, d, r, E, lens, "uniform", scale=2.0, seed=60 + d),
                                 "cuda", expert_ids=ids) for d in (264, 4112, 48, 4104)]
    for i in ins[1:]:
        i.x.copy_(ins[0].x)
    ctx = moin.Context(0)
    try:
        plan = moin.Plan(ctx)
        plan.build(ins[0].seq_offsets, ins[0].expert_ids, T, E)
        print(f"[gpu] decode stream, slabs and tiles in one call, d_in={d_in} r={r}", flush=True)
        for pick in (ins, ins[1:3], ins[:2]):
            ctx.timing_enable(True)
            ctx.timing_reset()
            ys = moin.moin_lora_linear_planned_shared(ctx, plan, pick[0].x, [i.W for i in pick], [i.A_stack for i in pick],
                                                      [i.B_stack for i in pick], 2.0)
            ctx.check()
            n = [ctx.timing_read(k)[1] for k in (moin.K_DECODE_SHRINK, moin.K_DECODE_EXPAND)]
            ctx.timing_enable(False)
            for y, i in zip(ys, pick):
                one = moin.moin_lora_linear_planned(ctx, plan, pick[0].x, i.W, i.A_stack, i.B_stack, 2.0)
                assert torch.equal(y.view(torch.int16), one.view(torch.int16))
            ctx.check()
            assert n == [1, 1], n
        plan.close()
    finally:
        ctx.close()


# base-only tokens (no adapter, or one of rank 0) have a pass of their own: none, some and nothing but them, rows of one
# and several pieces of 512 columns, ragged; parts of the base product from one to four, and rows by token (T > 1024)
@pytest.mark.parametrize("share", [1.0, 0.5, 0.02])
@pytest.mark.parametrize("T,E,d_in,d_out,r", [(5, 9, 256, 520, 64), (40, 9, 2048, 1032, 16), (70, 200, 5632, 488, 128),
                                              (300, 9, 4096, 8, 40), (1300, 700, 2048, 1544, 128)])
def test_base_only_tokens(T, E, d_in, d_out, r, share):
    rng = np.random.default_rng(T + d_out)
    lens = [1] * T
    ids = rng.integers(0, E, size=T).astype(np.int32)
    at = rng.random(T)
    ids[at < share / 2] = -1
    ranks = 8 * rng.integers(1, r // 8 + 1, size=E).astype(np.int32)
    ranks[np.unique(ids[(at < share) & (ids >= 0)])] = 0
    w = wl.LinearWorkload("base_only", d_in, d_out, r, E, lens, "uniform", scale=2.0, seed=T)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    rk = torch.from_numpy(ranks).cuda()
    ref = _reference(inp, ids, lens, rk, r)
    print(f"[gpu] base-only tokens T={T} {d_in}->{d_out} share={share}", flush=True)
    for dt in (torch.float32, torch.bfloat16):
        y = torch.full((T, d_out), float("nan"), dtype=dt, device="cuda")
        moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              rank_of_expert=rk, out=y, y_dtype=dt)
        gc.ctx().check()
        if dt == torch.float32:
            _check(y, ref, d_in, r)
        else:   # rounded to nearest: half an ulp (2^-9) of each value, beside the fp32 result's own bound
            slack = 4 * (d_in ** 0.5 + 128) * 2.0 ** -24 * float(ref.abs().max())
            assert bool(((y.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + slack).all())


def test_base_only_tokens_of_several_projections():
    T, E, d_in, r = 90, 9, 512, 32
    lens = [1] * T
    ids, ranks = _batch(lens, E, T)
    ids[::2] = -1
    ins = [wl.make_linear_inputs(wl.LinearWorkload("base_only", d_in, d, r, E, lens, "uniform", scale=2.0, seed=70 + d),
                                 "cuda", expert_ids=ids) for d in (1032, 8, 520)]
    for i in ins[1:]:
        i.x.copy_(ins[0].x)
    rk = ranks(r)
    plan = moin.Plan(gc.ctx())
    plan.build(ins[0].seq_offsets, ins[0].expert_ids, T, E, rank_of_expert=rk)
    print("[gpu] base-only tokens, three projections", flush=True)
    ys = moin.moin_lora_linear_planned_shared(gc.ctx(), plan, ins[0].x, [i.W for i in ins], [i.A_stack for i in ins],
                                              [i.B_stack for i in ins], 2.0, y_dtype=torch.float32)
    gc.ctx().check()
    for y, i in zip(ys, ins):
        _check(y, _reference(i, ids, lens, rk, r), d_in, r)
