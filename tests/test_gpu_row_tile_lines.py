"""Batches of short sequences on the lines between row tiles and tokens gathered by expert: rows that are not whole blocks in
half-empty row tiles beyond a round of the chip; against torch in fp64."""
import pytest
import torch

from paper_2410_09687_amd import moin
from tests import gpu_common as gc
from tests.test_gpu_both_groupings import E, _batch, _counted
from tests.test_gpu_decode_stream import _check, _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,d_in,d_out,r", [([80] * 40, 1000, 2048, 48), ([64] * 64, 1000, 2000, 64), ([64, 65, 127, 128, 1] * 20, 1000, 2048, 128),
                                               ([128, 129] * 21, 72, 2056, 16), ([100] * 24, 1416, 5632, 64)])
def test_rows_of_no_whole_blocks_in_half_empty_tiles(lens, d_in, d_out, r):
    inp, ids, rk = _batch(lens, d_in, d_out, r, len(lens) % 8 == 0)
    print(f"[gpu] half-empty row tiles T={sum(lens)} S={len(lens)} {d_in}->{d_out} r={r}", flush=True)
    ctx = gc.ctx()
    plan = moin.Plan(ctx).build(inp.seq_offsets, inp.expert_ids, sum(lens), E, rank_of_expert=rk)
    y = moin.moin_lora_linear_planned(ctx, plan, inp.x, inp.W, inp.A_stack, inp.B_stack, 2.0, y_dtype=torch.float32)
    ctx.check()
    _check(y, _reference(inp, ids, lens, rk, r), d_in, r)
    plan.close()


def _dequantised(codes, scales):   # E4M3 codes times 2^(scale - 127), the scale bytes of a row's 128 values side by side
    e = scales.permute(1, 0, 2).reshape(codes.shape[0], -1).repeat_interleave(32, dim=1)
    return codes.view(torch.float8_e4m3fn).double() * torch.exp2(e.double() - 127)


@pytest.mark.parametrize("lens,d_in,d_out,r,tiles", [
    ([500, 524], 3200, 200, 64, False), ([500, 525], 3200, 200, 64, True), ([768], 3072, 2048, 64, True), ([768], 3200, 200, 128, True),
    ([703], 2048, 256, 64, False), ([704], 2048, 256, 64, True), ([703], 2048, 392, 64, True), ([527], 2048, 200, 128, False),
    ([527], 1920, 200, 128, True), ([528], 2048, 200, 128, True)])
def test_lines_of_the_quantised_base(lens, d_in, d_out, r, tiles):
    inp, ids, _ = _batch(lens, d_in, d_out, r, False)
    print(f"[gpu] lines of the quantised base T={sum(lens)} S={len(lens)} {d_in}->{d_out} r={r}", flush=True)
    ctx = gc.ctx()
    Wq, Ws = moin.moin_mx_quantize(ctx, inp.W, blocked=True)
    xq, xs = moin.moin_mx_quantize(ctx, inp.x, blocked=True)
    plan = moin.Plan(ctx).build(inp.seq_offsets, inp.expert_ids, sum(lens), E)
    y, took = _counted(ctx, lambda: moin.moin_lora_linear_mx_planned(ctx, plan, inp.x, Wq, Ws, inp.A_stack, inp.B_stack, 2.0,
                                                                     y_dtype=torch.float32))
    assert took == tiles
    on_x = _reference(inp, ids, lens, None, r) - inp.x.double() @ inp.W.double().T   # the adapters' share
    _check(y, on_x + _dequantised(xq, xs) @ _dequantised(Wq, Ws).T, d_in, r)
    plan.close()
