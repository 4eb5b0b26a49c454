"""Routing launches that sum the centroids' norms on their way: the ids, and the norms they leave for later calls, are those of
the call with the norms computed ahead; K around a tile and a multiple of 256, every number of blocks, retained slots, a
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
