"""The kernels that serve batches beyond the chip's first round of small tiles, at their edges: row counts around a tile, output
tails of 8, contraction lengths and ranks inside a block, experts of smaller rank and of none, sequences without an adapter,
fp32 and bf16 results; against torch in fp64.  Each test first asserts that its batch lies beyond the small tiles' rule."""
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


def _inputs(lens, ids, d_in, d_out, r, seed):
    w = wl.LinearWorkload("large", d_in, d_out, r, E, lens, "uniform", scale=2.0, seed=seed)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    inp.A_stack[4] = float("nan")   # (no sequence uses it)
    inp.B_stack[4] = float("nan")
    return inp


def _own_ranks(inp, r, ranked):
    """Own ranks, one of them 0; what must not be read is NaN (B_e up to the end of a block of 64 meets zeros)."""
    if not ranked:
        return None
    ranks = [r, 8, max(8, r - 8), 0, 8]
    for e, k in enumerate(ranks):
        inp.A_stack[e, k:] = float("nan")
        inp.B_stack[e, :, k:] = float("nan")
        inp.B_stack[e, :, k:(k + 63) // 64 * 64] = 0
    inp.A_stack[4] = float("nan")
    return torch.tensor(ranks, dtype=torch.int32, device="cuda")


def _beyond(lens, rows, columns, per_unit):
    """The batch's tiles of `rows` tokens, its sequences taken to be of equal length, times `columns`: more than the rule's."""
    n = len(lens) * -(-(-(-sum(lens) // len(lens))) // rows) * columns
    assert n > per_unit * torch.cuda.get_device_properties(0).multi_processor_count


def _compare(y, ref, d_in, r):
    if y.dtype == torch.float32:
        _check(y, ref, d_in, r)
    else:   # rounded to bf16: half a unit of the last of 8 bits
        assert bool(((y.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all())


def _clean(inp):
    """NaN would reach the reference through the columns it leaves out."""
    return wl.LinearInputs(inp.wl, inp.x, inp.W, inp.A_stack.nan_to_num(0), inp.B_stack.nan_to_num(0), inp.seq_offsets,
                           inp.expert_ids)


@pytest.mark.parametrize("d_in,d_out,r,ranked,f32", [
    (72, 2056, 24, True, True), (200, 2056, 40, False, False), (1000, 2040, 136, True, True), (328, 3336, 72, True, False),  # tiles through registers
    (192, 2056, 24, True, True), (128, 2056, 64, True, False), (320, 2040, 136, True, True), (256, 3336, 72, False, False)])  # streaming
def test_prefill(d_in, d_out, r, ranked, f32):
    lens, ids = LENS * 4, np.tile(IDS, 4)
    _beyond(lens, 128, -(-d_out // 128), 2)
    inp = _inputs(lens, ids, d_in, d_out, r, d_in + r)
    rk = _own_ranks(inp, r, ranked)
    print(f"[gpu] large prefill {d_in}->{d_out} r={r} ranked={ranked} f32={f32}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32 if f32 else torch.bfloat16, rank_of_expert=rk)
    gc.ctx().check()
    _compare(y, _reference(_clean(inp), ids, lens, rk, r), d_in, r)


@pytest.mark.parametrize("d_in,r,widths", [(256, 24, (2056, 136, 8)), (192, 136, (264, 2040))])
def test_prefill_shared(d_in, r, widths):
    lens, ids = LENS * 4, np.tile(IDS, 4)
    _beyond(lens, 128, sum(-(-d // 128) for d in widths), 2)
    ins = [_inputs(lens, ids, d_in, d, r, 60 + d) for d in widths]
    for i in ins[1:]:
        i.x.copy_(ins[0].x)
    rk = [_own_ranks(i, r, True) for i in ins][0]
    plan = moin.Plan(gc.ctx()).build(ins[0].seq_offsets, ins[0].expert_ids, sum(lens), E, rank_of_expert=rk)
    print(f"[gpu] large prefill shared d_in={d_in} r={r} {widths}", flush=True)
    ys = moin.moin_lora_linear_planned_shared(gc.ctx(), plan, ins[0].x, [i.W for i in ins], [i.A_stack for i in ins],
                                              [i.B_stack for i in ins], 2.0, y_dtype=torch.float32)
    gc.ctx().check()
    for y, i in zip(ys, ins):
        _check(y, _reference(_clean(i), ids, lens, rk, r), d_in, r)
    plan.close()


@pytest.mark.parametrize("d_in,r", [(72, 24), (200, 40), (1000, 0), (192, 16), (256, 0)])
@pytest.mark.parametrize("f32", [True, False])
def test_gathered(d_in, r, f32):
    S, d_out = 5001, 2056
    _beyond([S], 128, -(-d_out // 128), 2)   # plain row tiles
    ids = (np.arange(S) % E - 1 if r else np.full(S, -1)).astype(np.int32)   # -1 .. 3
    inp = _inputs([1] * S, ids, d_in, d_out, max(r, 8), d_in + r)
    A, B = (inp.A_stack, inp.B_stack) if r else (None, None)
    print(f"[gpu] large gathered batch d_in={d_in} r={r} f32={f32}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, A, B, 2.0,
                              y_dtype=torch.float32 if f32 else torch.bfloat16)
    gc.ctx().check()
    _compare(y, _reference(inp, ids, [1] * S, None, r), d_in, max(r, 8))


@pytest.mark.parametrize("d_in,r,times", [(64, 24, 10), (192, 32, 10), (320, 64, 10), (192, 72, 14), (704, 128, 10), (128, 136, 1)])
def test_shrink(d_in, r, times):
    lens, ids = LENS * times, np.tile(IDS, times)
    if r <= 128:
        _beyond(lens, 32, 1 if r <= 32 else -(-r // 32), 3 if r <= 32 else 4 if r <= 64 else 12)
    inp = _inputs(lens, ids, d_in, 8, r, d_in + r)
    rk = _own_ranks(inp, r, True)
    print(f"[gpu] shrink of many row tiles d_in={d_in} r={r}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32, rank_of_expert=rk)
    gc.ctx().check()
    _check(y, _reference(_clean(inp), ids, lens, rk, r), d_in, r)


# ---- quantised base ----

def _mx_base(x, W):
    """x W^T of the quantised values, in fp64."""
    def values(t):
        codes, scales = moin.moin_mx_quantize(gc.ctx(), t)
        v = codes.view(torch.float8_e4m3fn).double().view(t.shape[0], -1, 32)
        return (v * torch.exp2(scales.double() - 127).unsqueeze(2)).view(t.shape)
    return values(x) @ values(W).T


def _mx_reference(inp, ids, lens, rk, r):
    c = _clean(inp)
    term = _reference(wl.LinearInputs(c.wl, c.x, torch.zeros_like(c.W), c.A_stack, c.B_stack, c.seq_offsets, c.expert_ids),
                      ids, lens, rk, r)
    return _mx_base(inp.x, inp.W) + term


@pytest.mark.parametrize("d_in,d_out,r,ranked,f32", [
    (256, 2056, 64, True, True), (640, 2040, 128, True, False), (384, 3336, 192, True, True), (256, 2184, 128, False, True)])
def test_quantised_prefill(d_in, d_out, r, ranked, f32):
    lens, ids = LENS * 4, np.tile(IDS, 4)
    _beyond(lens, 128, -(-d_out // 128), 2)
    inp = _inputs(lens, ids, d_in, d_out, r, d_in + r)
    rk = _own_ranks(inp, r, ranked)
    Wq, Ws = moin.moin_mx_quantize(gc.ctx(), inp.W, blocked=True)
    print(f"[gpu] large quantised prefill {d_in}->{d_out} r={r} ranked={ranked} f32={f32}", flush=True)
    y = moin.moin_lora_linear_mx(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, Wq, Ws, inp.A_stack, inp.B_stack, 2.0,
                                 y_dtype=torch.float32 if f32 else torch.bfloat16, rank_of_expert=rk)
    gc.ctx().check()
    _compare(y, _mx_reference(inp, ids, lens, rk, r), d_in, r)


@pytest.mark.parametrize("d_in,r", [(256, 64), (640, 128), (512, 0)])
def test_quantised_gathered(d_in, r):
    S, d_out = 5001, 2056
    _beyond([S], 128, -(-d_out // 128), 2)
    ids = (np.arange(S) % E - 1 if r else np.full(S, -1)).astype(np.int32)
    inp = _inputs([1] * S, ids, d_in, d_out, max(r, 64), d_in + r)
    A, B = (inp.A_stack, inp.B_stack) if r else (None, None)
    Wq, Ws = moin.moin_mx_quantize(gc.ctx(), inp.W, blocked=True)
    print(f"[gpu] large quantised gathered batch d_in={d_in} r={r}", flush=True)
    y = moin.moin_lora_linear_mx(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, Wq, Ws, A, B, 2.0, y_dtype=torch.float32)
    gc.ctx().check()
    _check(y, _mx_reference(inp, ids, [1] * S, None, r), d_in, max(r, 64))


@pytest.mark.parametrize("d_in,r,times", [(256, 64, 6), (384, 128, 6), (256, 192, 1)])
def test_quantising_shrink(d_in, r, times):
    lens, ids, ctx = LENS * times, np.tile(IDS, times), gc.ctx()
    if r <= 128:
        _beyond(lens, 32, -(-r // 32), 6 if r > 64 else 3)
    T = sum(lens)
    inp = _inputs(lens, ids, d_in, 72, r, d_in + r)
    rk = _own_ranks(inp, r, True)
    Wq, Ws = moin.moin_mx_quantize(ctx, inp.W, blocked=True)
    want_q, want_s = moin.moin_mx_quantize(ctx, inp.x, blocked=True)
    plan = moin.Plan(ctx).build(inp.seq_offsets, inp.expert_ids, T, E, rank_of_expert=rk)
    xq = torch.zeros((T, d_in), dtype=torch.uint8, device="cuda")
    xs = torch.zeros((d_in // 128, T, 4), dtype=torch.uint8, device="cuda")
    call = lambda **kw: moin.moin_lora_linear_mx_planned(ctx, plan, inp.x, Wq, Ws, inp.A_stack, inp.B_stack, 2.0,
                                                         y_dtype=torch.float32, **kw)
    print(f"[gpu] quantising shrink of many row tiles d_in={d_in} r={r}", flush=True)
    made, given = call(xq=xq, xs=xs, emit=True), call(xq=xq, xs=xs)
    ctx.check()
    assert torch.equal(xq, want_q.view(torch.uint8)) and torch.equal(xs, want_s) and torch.equal(made, given)
    _check(made, _mx_reference(inp, ids, lens, rk, r), d_in, r)
    plan.close()
