"""Routing launches that sum the centroids' norms on their way: the ids, and the bits of the norms (also those they leave for
later calls), are those of the call with the norms computed ahead; K around a tile and a multiple of 256, every number of blocks, retained slots, a
second call that vouches for the table, one that changes it, huge and undefined centroids."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,D", [(1, 1, 64), (3, 63, 128), (64, 64, 192), (65, 65, 256), (130, 255, 384), (7, 256, 768), (9, 257, 320),
                                   (512, 500, 768), (700, 300, 1024), (4096, 100, 64)])
@pytest.mark.parametrize("retained", [False, True])
def test_same_ids_and_norms(N, K, D, retained):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + K + D)
    cent = torch.randn((K, D), device="cuda", generator=g).bfloat16()
    emb = (cent[torch.randint(0, K, (N,), device="cuda", generator=g)].float() + torch.randn((N, D), device="cuda", generator=g)).bfloat16()
    slot = torch.from_numpy(np.where(np.arange(K) % 3 == 1, -1, np.arange(K)).astype(np.int32)).cuda()
    ctx = gc.ctx()
    print(f"[gpu] norms in the routing launch N={N} K={K} D={D} retained={retained}", flush=True)
    call = lambda c, **kw: moin.moin_route(ctx, emb, c, slot, retained_only=retained, want_counts=True, **kw)
    here = call(cent)                             # norms computed on the way
    vouched = call(cent, same_centroids=True)     # the norms it left
    ahead = call(cent, static=True)               # a launch of its own for them
    other = call(cent * 0.5)                      # another table
    again = call(cent)
    ctx.check()
    for a, b in ((here, vouched), (here, ahead), (here, again)):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
    ok = None if not retained else (slot.cpu().numpy() >= 0)
    gc.check_route(emb, cent, here[1], eligible=ok)
    gc.check_route(emb, (cent * 0.5), other[1], eligible=ok)


def test_undefined_and_huge_centroids():
    emb = torch.randn((20, 128), device="cuda").bfloat16()
    cent = torch.randn((70, 128), device="cuda").bfloat16()
    cent[3], cent[64], cent[69] = float("nan"), float("inf"), 1e30   # squares that are no number, or infinite
    ctx = gc.ctx()
    a, b = (moin.moin_route(ctx, emb, cent, static=s) for s in (False, True))
    c = moin.moin_route(ctx, emb, cent, same_centroids=True)
    ctx.check()
    assert torch.equal(a[1], b[1]) and torch.equal(a[1], c[1])
    assert not bool(torch.isin(a[1], torch.tensor([3, 64, 69], device="cuda", dtype=torch.int32)).any())


def _norms(cent):
    """The sums of squares as the kernels make them: lane i of 64 its values i, i + 64, ... by fused multiply-adds, then lanes 32,
    16, ..., 1 apart, all in fp32 (a bf16 square has 16 bits, so the fused step is one rounding of an exact fp64 sum)."""
    v = cent.float().double().cpu().numpy().reshape(cent.shape[0], -1, 64)
    acc = np.zeros((cent.shape[0], 64), dtype=np.float32)
    for b in range(v.shape[1]):
        acc = (acc.astype(np.float64) + v[:, b] ** 2).astype(np.float32)
    o = 32
    while o:
        acc = acc + acc[:, np.arange(64) ^ o]
        o //= 2
    return acc[:, 0]


@pytest.mark.parametrize("K,D,N,large", [(48, 64, 1, 8), (64, 192, 3, 4), (70, 768, 65, 4)])
def test_the_norms_to_the_last_bit(K, D, N, large):
    # Centroids that are permutations of each other: their norms differ by the rounding of the sums alone.  For a query of
    # zeros the nearest is the one of the smallest norm, the lowest index among equals; taken out one after the other they
    # come in the order of the norms' bits.
    rng = np.random.default_rng(K + D)
    row = rng.normal(size=D) * np.where(rng.random(D) < 0.05, large, 1)   # (a few large values: more to round)
    cent = torch.from_numpy(np.stack([rng.permutation(row) for _ in range(K)])).cuda().bfloat16()
    norms = _norms(cent)
    want = np.lexsort((np.arange(K), norms))
    exact = (cent.float().double().cpu().numpy() ** 2).sum(1)
    assert np.ptp(exact) < 1e-9 and len(np.unique(norms)) >= 3 and not np.array_equal(want, np.arange(K))
    emb = torch.zeros((N, D), device="cuda", dtype=torch.bfloat16)
    slot = torch.arange(K, dtype=torch.int32, device="cuda")
    ctx, got = gc.ctx(), ([], [], [])
    print(f"[gpu] norms bit by bit K={K} D={D} N={N}", flush=True)
    for k in want:
        here = moin.moin_route(ctx, emb, cent, slot, retained_only=True)                          # on the way
        left = moin.moin_route(ctx, emb, cent, slot, retained_only=True, same_centroids=True)     # the norms it left
        ahead = moin.moin_route(ctx, emb, cent, slot, retained_only=True, static=True)            # a launch of their own
        for g, r in zip(got, (here, left, ahead)):
            assert bool((r[1] == r[1][0]).all())
            g.append(int(r[1][0]))
        slot[int(k)] = -1
    ctx.check()
    assert got[0] == got[1] == got[2] == want.tolist()


@pytest.mark.parametrize("N,K,D", [(1024, 1024, 448), (1025, 1024, 448), (1025, 1024, 384)])
def test_either_side_of_the_line_for_long_sums(N, K, D):   # a tile per compute unit, more, more of short sums
    test_same_ids_and_norms(N, K, D, True)
