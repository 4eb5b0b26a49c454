"""An eager call with the largest batch prepares the captured calls of batches of no more sequences and tokens: those that
take the other grouping, whose base product is cut into more parts, or whose projections share their launches."""
import pytest
import torch

from paper_2410_09687_amd import moin
from tests import gpu_common as gc
from tests.test_gpu_both_groupings import E, _batch

pytestmark = pytest.mark.gpu


def _call(ctx, kind, plan, inp, outs=None):
    """One call of the kind, on one projection or on two of the same width; its outputs."""
    if kind == "shared":
        return moin.moin_lora_linear_planned_shared(ctx, plan, inp.x, [inp.W] * 2, [inp.A_stack] * 2, [inp.B_stack] * 2, 2.0, outs=outs)
    out = outs[0] if outs else None
    if kind == "mx":
        return [moin.moin_lora_linear_mx_planned(ctx, plan, inp.x, *inp.quantised, inp.A_stack, inp.B_stack, 2.0, out=out)]
    return [moin.moin_lora_linear_planned(ctx, plan, inp.x, inp.W, inp.A_stack, inp.B_stack, 2.0, out=out)]


@pytest.mark.parametrize("first,then,d_in,d_out,r", [
    ([1] * 1100, [1] * 1000, 5632, 2048, 128),     # plain row tiles / four parts
    ([128] * 9, [330], 2048, 2048, 16),            # row tiles or gathered by the call
    ([500, 524], [300], 2048, 2048, 64),
    ([1100, 900], [700, 500], 2048, 264, 64),      # row tiles both
    ([897], [896], 4096, 4096, 16),                # two parts / three
    ([1] * 1024, [1] * 896, 2048, 8192, 64),       # one part / two
    ([1] * 9000, [1] * 8000, 1000, 256, 32),       # whole / parts of rows that are not whole blocks
    ([64] * 256, [16000], 2048, 8, 8),             # gathered / row tiles, whose rows of u are padded to 64
    ([1] * 300, [1] * 128, 2048, 2048, 128)])
@pytest.mark.parametrize("kind", ["plain", "shared", "mx"])
def test_captured_after_the_largest_eager_call(first, then, d_in, d_out, r, kind):
    if kind == "mx" and (r % 64 or d_in % 128):
        pytest.skip("not a shape of the quantised base")
    ctx = moin.Context(0)
    try:
        for lens in (first, then):
            inp, _, _ = _batch(lens, d_in, d_out, r, False)
            plan = moin.Plan(ctx).build(inp.seq_offsets, inp.expert_ids, sum(lens), E)
            if kind == "mx":
                inp.quantised = moin.moin_mx_quantize(ctx, inp.W, blocked=True)
            if lens is first:
                _call(ctx, kind, plan, inp)
                ctx.check()
                size = ctx.workspace_bytes()
                plan.close()
        print(f"[gpu] captured {kind} {len(then)} sequences, {sum(then)} tokens after {sum(first)}, {d_in}->{d_out} r={r}", flush=True)
        outs = [torch.empty((sum(then), d_out), dtype=torch.bfloat16, device="cuda") for _ in range(2 if kind == "shared" else 1)]
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _call(ctx, kind, plan, inp, outs)
        other = gc.ctx()
        other_plan = moin.Plan(other).build(inp.seq_offsets, inp.expert_ids, sum(then), E)
        eager = _call(other, kind, other_plan, inp)
        other.check()
        for _ in range(2):
            for y in outs:
                y.fill_(float("nan"))
            graph.replay()
            ctx.check()
            for y, want in zip(outs, eager):
                assert torch.equal(y.view(torch.int16), want.view(torch.int16))
        assert ctx.workspace_bytes() == size
        del graph
        other_plan.close()
        plan.close()
    finally:
        torch.cuda.synchronize()
        ctx.close()


@pytest.mark.parametrize("first,then", [([68] * 16 + [12], [62] * 16), ([300] * 4, [100] * 4), ([9000], [128]), ([1] * 4100, [1] * 4096),
                                        ([2048, 2048, 300], [1023, 1])])
def test_smaller_batches_are_grouped_under_capture(first, then):
    ctx, other = moin.Context(0), gc.ctx()
    try:
        plan = moin.Plan(ctx)
        inp, _, _ = _batch(first, 128, 72, 16, False)
        plan.build(inp.seq_offsets, inp.expert_ids, sum(first), E)
        ctx.reserve_workspace(8 << 20)
        inp, _, _ = _batch(then, 128, 72, 16, False)
        eager = _call(other, "plain", moin.Plan(other).build(inp.seq_offsets, inp.expert_ids, sum(then), E), inp)[0]
        out = torch.empty_like(eager)
        print(f"[gpu] captured grouping of {len(then)} sequences, {sum(then)} tokens after {sum(first)}", flush=True)
        ctx.check()
        other.check()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            plan.build(inp.seq_offsets, inp.expert_ids, sum(then), E)
            _call(ctx, "plain", plan, inp, [out])
        for _ in range(2):
            out.fill_(float("nan"))
            graph.replay()
            ctx.check()
            assert torch.equal(out.view(torch.int16), eager.view(torch.int16))
        del graph
        plan.close()
    finally:
        torch.cuda.synchronize()
        ctx.close()
