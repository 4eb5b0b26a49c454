"""The grouping where a sequence's tokens are written by a thread, by eight lanes and by a wave (8 / 9 and 256 / 257 tokens), a
group's records by a thread and by a wave (4 / 5 records), and the sequences compared sixteen at a time (15 to 17, 127 to
129): every token's output against torch in fp64, the grouping in a launch of its own and behind the routing."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc
from tests.test_gpu_decode_stream import _check, _reference
from tests.test_gpu_plan_sizes import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [15, 16, 17, 64, 127, 128, 129, 600])
def test_lengths_and_records(S):
    rng = np.random.default_rng(S)
    lens = rng.choice([0, 1, 7, 8, 9, 15], size=S)
    lens[:6] = [256, 257, 300, 8, 9, 3]    # on average fewer than 64 tokens: gathered
    _run(S, 3, lens, S, ranked=S % 2 == 1)   # three experts: groups of many records, base-only ones among them


@pytest.mark.parametrize("S", [1, 16, 100, 300, 512])
def test_behind_the_routing(S):
    rng = np.random.default_rng(S)
    K, E, D = 40, 7, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(S)
    emb, cent = (torch.randn((n, D), device="cuda", generator=g).bfloat16() for n in (S, K))
    slot = torch.from_numpy(np.where(np.arange(K) < E, np.arange(K), -1).astype(np.int32)).cuda()
    lens = rng.choice([1, 8, 9, 70], size=S)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    T, d_in, d_out, r = int(lens.sum()), 128, 72, 16
    x, W = torch.randn((T, d_in), device="cuda", generator=g).bfloat16(), torch.randn((d_out, d_in), device="cuda", generator=g).bfloat16()
    A, B = (torch.randn(s, device="cuda", generator=g).bfloat16() for s in ((E, r, d_in), (E, d_out, r)))
    ranks = torch.tensor([16, 8, 0, 16, 8, 16, 8], dtype=torch.int32, device="cuda")
    ctx, ys = gc.ctx(), []
    for fused in (True, False):
        plan = moin.Plan(ctx)
        if fused:
            eids, _, _ = moin.moin_route_plan(ctx, plan, emb, cent, off, T, E, slot, rank_of_expert=ranks)
        else:
            eids, _, _ = moin.moin_route(ctx, emb, cent, slot)
            plan.build(off, eids, T, E, rank_of_expert=ranks)
        ys.append(moin.moin_lora_linear_planned(ctx, plan, x, W, A, B, 2.0, y_dtype=torch.float32))
        ctx.check()
        plan.close()
    assert torch.equal(ys[0], ys[1])
    tok = torch.repeat_interleave(eids.long(), torch.from_numpy(lens).cuda())
    ref = x.double() @ W.double().T
    for e in range(E):
        at, k = (tok == e).nonzero()[:, 0], int(ranks[e])
        ref[at] += 2.0 * (x[at].double() @ A[e, :k].double().T) @ B[e, :, :k].double().T
    # sums of 128 + 16 products in fp32 and u as a bf16 pair: 2e-5 of the largest output holds
    assert float((ys[0].double() - ref).abs().max()) <= 2e-5 * float(ref.abs().max())


# Tokens per expert, cut into records of 16 (up to 1024 tokens) or 128 (beyond 16 384): eight and nine records more than groups;
# eight and nine groups of five; more than eight groups, one of 64 and one of 65; lengths of a sequence.
@pytest.mark.parametrize("groups,length", [([144, 1, 1], 9), ([145, 1, 1], 9), ([80] * 8, 5), ([80] * 9, 5), ([16] * 8 + [33], 1), ([7], 1),
                                           ([8192] * 9 + [8193], 48), ([8192, 8193, 600], 30), ([70] * 12, 1)])
def test_records_of_few_and_many_groups(groups, length):
    lens, ids = [], []
    for e, n in enumerate(groups):
        cut = [length] * (n // length) + ([n % length] if n % length else [])
        lens += cut
        ids += [e - 1] * len(cut)          # (the first group without an adapter)
    at = np.random.default_rng(len(lens)).permutation(len(lens))
    lens, ids = [lens[i] for i in at], np.array(ids, dtype=np.int32)[at]
    d_in, r, E = 128, 16, len(groups)
    inp = wl.make_linear_inputs(wl.LinearWorkload("records", d_in, 72, r, E, lens, "uniform", scale=2.0, seed=len(lens)), "cuda",
                                expert_ids=ids)
    print(f"[gpu] records of {len(groups)} groups, S={len(lens)} T={sum(lens)}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32)
    gc.ctx().check()
    _check(y, _reference(inp, ids, lens, None, r), d_in, r)
