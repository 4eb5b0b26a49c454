"""The grouping of a batch at the sizes where its sort changes (comparison up to 128 sequences, radix in LDS up to
12288, one radix digit of seven bits more with the number of experts, bitonic through memory beyond): every token's
output against torch in fp64, through the decode / gather kernels and through the prefill tiles."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu

D_IN, D_OUT, R = 128, 72, 16


def _run(S, E, lens, seed, ranked):
    rng = np.random.default_rng(seed)
    T = int(lens.sum())
    ids = rng.integers(-1, E, size=S).astype(np.int32)
    ids[rng.random(S) < 0.3] = E - 1               # a hot expert, and the largest key
    w = wl.LinearWorkload("plan", D_IN, D_OUT, R, E, lens.tolist(), "uniform", scale=2.0, seed=seed)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    ranks = torch.from_numpy((8 * rng.integers(0, R // 8 + 1, size=E)).astype(np.int32)).cuda() if ranked else None
    print(f"[gpu] plan S={S} E={E} T={T} ranked={ranked}", flush=True)
    y = moin.moin_lora_linear(gc.ctx(), inp.x, inp.seq_offsets, inp.expert_ids, inp.W, inp.A_stack, inp.B_stack, 2.0,
                              y_dtype=torch.float32, rank_of_expert=ranks)
    gc.ctx().check()
    tok = torch.from_numpy(np.repeat(ids, lens).astype(np.int64)).cuda()
    x = inp.x.double()
    u = torch.zeros((T, R), dtype=torch.float64, device="cuda")
    ref = x @ inp.W.double().T
    for lo in range(0, T, 8192):                   # (per-token adapters, a slab at a time)
        t = tok[lo:lo + 8192]
        e = t.clamp(min=0)
        u = (inp.A_stack[e].double() * x[lo:lo + 8192, None, :]).sum(2)
        u[t < 0] = 0
        if ranks is not None:
            u[torch.arange(R, device="cuda")[None] >= ranks[e][:, None]] = 0
        ref[lo:lo + 8192] += 2.0 * (inp.B_stack[e].double() * u[:, None, :]).sum(2)
    # bf16 products are exact in fp32; sums of 128 + 16 terms and u as a bf16 pair: 2e-5 of the largest output holds
    assert float((y.double() - ref).abs().max()) <= 2e-5 * float(ref.abs().max())


@pytest.mark.parametrize("S,E", [(1, 1), (2, 3), (127, 50), (128, 5000), (129, 127), (129, 128), (512, 16383),
                                 (513, 16384), (2049, 300), (8192, 5000), (12288, 700), (12289, 700)])
def test_grouping_of_short_sequences(S, E):
    rng = np.random.default_rng(S + E)
    lens = rng.choice([0, 1, 1, 2, 9, 40] if S < 4000 else [0, 1, 1, 2], size=S)
    lens[-1] = 1
    _run(S, E, lens, 5 * S + E, ranked=S % 2 == 1)


@pytest.mark.parametrize("S,E", [(1, 2), (60, 9), (130, 40), (520, 200)])
def test_grouping_into_prefill_tiles(S, E):
    rng = np.random.default_rng(S + E)
    lens = rng.integers(100, 300, size=S)
    lens[0] = 1300
    _run(S, E, lens, 7 * S + E, ranked=S % 2 == 0)
