"""The update's sort in one launch: points around a wave's run, centres around a thread's, one heavy centre and all in one,
empty centres, ids out of range; against the update on a table of more points (the launches of the larger sort) and numpy."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(1, 1), (2, 7), (63, 64), (513, 511), (1000, 513), (4097, 6144), (4097, 6145), (5120, 5000),
                                 (5120, 3), (5121, 3)])
@pytest.mark.parametrize("how", ["even", "heavy", "one"])
def test_against_numpy(N, K, how):
    rng = np.random.default_rng(N + K)
    D = 64
    x = torch.from_numpy(rng.integers(-8, 9, size=(N, D)).astype(np.float32)).cuda()   # sums are exact in any order
    ids = {"even": rng.integers(0, K, size=N), "heavy": np.where(rng.random(N) < 0.7, K // 2, rng.integers(0, K, size=N)),
           "one": np.full(N, K - 1)}[how].astype(np.int32)
    cent = torch.from_numpy(rng.integers(-8, 9, size=(K, D)).astype(np.float32)).cuda()
    print(f"[gpu] kmeans sort N={N} K={K} {how}", flush=True)
    new, counts, inertia = moin.moin_kmeans_update(gc.ctx(), x, torch.from_numpy(ids).cuda(), cent)
    gc.ctx().check()
    n = np.bincount(ids, minlength=K)
    assert np.array_equal(counts.cpu().numpy(), n)
    xs, c = x.cpu().numpy().astype(np.float64), cent.cpu().numpy().astype(np.float64)
    sums = np.zeros((K, D))
    np.add.at(sums, ids, xs)
    ref = np.where(n[:, None] > 0, sums / np.maximum(n, 1)[:, None], c).astype(np.float32)
    assert np.array_equal(new.cpu().numpy(), ref)
    assert float(inertia) == float(((xs - c[ids]) ** 2).sum())   # whole numbers below 2^53


def test_repeats_and_follows_the_order_of_the_points():
    rng = np.random.default_rng(5)
    N, K, D = 5000, 30, 128
    x = torch.from_numpy(rng.standard_normal((N, D)).astype(np.float32)).cuda()
    ids = torch.from_numpy(rng.integers(0, K, size=N).astype(np.int32)).cuda()
    cent = torch.zeros((K, D), device="cuda")
    a, b = (moin.moin_kmeans_update(gc.ctx(), x, ids, cent) for _ in range(2))
    # the same points with others behind them, beyond the one launch's limit: the same lists, hence the same bits
    more = torch.cat([x, x]), torch.cat([ids, torch.full((5000,), K, dtype=torch.int32, device="cuda")])
    c = moin.moin_kmeans_update(gc.ctx(), more[0], more[1], torch.zeros((K + 1, D), device="cuda"))
    gc.ctx().check()
    assert torch.equal(a[0], b[0]) and torch.equal(a[2], b[2])
    assert torch.equal(a[0], c[0][:K]) and torch.equal(a[1], c[1][:K])


def test_ids_out_of_range_are_left_out():
    ctx = moin.Context(0)
    x = torch.ones((300, 64), device="cuda")
    ids = torch.zeros(300, dtype=torch.int32, device="cuda")
    ids[7], ids[100], ids[299] = -1, 5, 1 << 30
    new, counts, _ = moin.moin_kmeans_update(ctx, x, ids, torch.zeros((5, 64), device="cuda"))
    assert counts.tolist() == [297, 0, 0, 0, 0] and bool((new[0] == 1).all()) and bool((new[1:] == 0).all())
    with pytest.raises(moin.MoinError):
        ctx.check()
    ctx.close()
