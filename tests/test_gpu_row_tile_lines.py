"""Batches of short sequences on the lines between row tiles and tokens gathered by expert: rows that are not whole blocks in
half-empty row tiles beyond a round of the chip; against torch in fp64."""
import pytest
import torch

from paper_2410_09687_amd import moin
from tests import gpu_common as gc
from tests.test_gpu_both_groupings import E, _batch
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
