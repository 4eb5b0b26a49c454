"""The decode base product at the edges of the rule for its parts: 32 / 33 and 128 / 129 tokens, contractions that end
inside a part or a block, one to four parts, rows that go through registers, slabs beside tiles in a shared call; against
torch in fp64."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc
from tests.test_gpu_decode_stream import _check, _reference

pytestmark = pytest.mark.gpu
E = 5


@pytest.mark.parametrize("T", [32, 33, 128, 129])
@pytest.mark.parametrize("d_in,r,ranked", [(256, 16, False), (320, 8, True), (1000, 64, False), (1088, 40, False), (2048, 128, True),
                                           (2112, 136, False), (5632, 32, False)])
def test_parts(T, d_in, r, ranked):
    lens = [T // 4 - 3, 7, T - T // 4 - 9, 5]
    ids = np.array([1, -1, 3, 0], dtype=np.int32)
    w = wl.LinearWorkload("parts", d_in, 264, r, E, lens, "uniform", scale=2.0, seed=d_in + T)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    inp.A_stack[4] = float("nan")   # (no sequence uses it)
    inp.B_stack[4] = float("nan")
    rk = torch.tensor([r, 8, 0, max(8, r - 8), 8], dtype=torch.int32, device="cuda") if ranked else None
    print(f"[gpu] parts of the base product T={T} {d_in}->264 r={r} ranked={ranked}", flush=True)
    ctx = gc.ctx()
    plan = moin.Plan(ctx).build(inp.seq_offsets, inp.expert_ids, T, E, rank_of_expert=rk)
    # (8192 outputs: beyond what goes in slabs at 17 to 32 tokens, so that the call mixes the two)
    W2 = torch.cat([inp.W] * 32)[:8192].contiguous()
    B2 = torch.cat([inp.B_stack] * 32, dim=1)[:, :8192].contiguous()
    one = moin.moin_lora_linear_planned(ctx, plan, inp.x, inp.W, inp.A_stack, inp.B_stack, 2.0, y_dtype=torch.float32)
    two = moin.moin_lora_linear_planned_shared(ctx, plan, inp.x, [W2, inp.W], [inp.A_stack] * 2, [B2, inp.B_stack], 2.0,
                                               y_dtype=torch.float32)
    ctx.check()
    ref = _reference(inp, ids, lens, rk, r)
    _check(one, ref, d_in, r)
    _check(two[1], ref, d_in, r)
    _check(two[0], torch.cat([ref] * 32, dim=1)[:, :8192], d_in, r)
    plan.close()
