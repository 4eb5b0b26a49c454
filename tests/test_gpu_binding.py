"""The natively marshalled calls: what they refuse and as what, results in the caller's own tensors, generators and other
sequences as lists, the library's status as MoinError, streams, and results that outlive their inputs."""
import gc as pygc

import pytest
import torch

from paper_2410_09687_amd import moin
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu

BF, I32 = torch.bfloat16, torch.int32
T, DI, DO, R, E, K, D = 12, 64, 72, 8, 3, 5, 64


def _t(*shape, dtype=BF, device="cuda"):
    return torch.ones(shape, device=device).to(dtype)


@pytest.fixture
def s():
    ctx = gc.ctx()
    off = torch.tensor([0, 5, T], dtype=I32, device="cuda")
    ids = torch.tensor([2, -1], dtype=I32, device="cuda")
    plan = moin.Plan(ctx).build(off, ids, T, E)
    yield dict(ctx=ctx, off=off, ids=ids, plan=plan, x=_t(T, DI), W=_t(DO, DI), A=_t(E, R, DI), B=_t(E, DO, R),
               emb=_t(2, D), cent=_t(K, D))
    plan.close()


def _planned(s, **kw):
    a = {**s, **kw}
    return moin.moin_lora_linear_planned(a["ctx"], a["plan"], a["x"], a["W"], a["A"], a["B"], 2.0, y_dtype=a.get("y", BF),
                                         out=a.get("out"))


@pytest.mark.parametrize("kw,error", [
    (lambda: dict(x=_t(T, DI, device="cpu")), ValueError), (lambda: dict(x=_t(T, DI, dtype=torch.float32)), TypeError), (lambda: dict(x=_t(T + 1, DI)), ValueError),
    (lambda: dict(x=_t(DI)), ValueError), (lambda: dict(W=_t(DO, DI + 8)), ValueError), (lambda: dict(A=_t(E, R + 8, DI)), ValueError),
    (lambda: dict(B=_t(DO, R)), ValueError), (lambda: dict(A=_t(E, R, DI, dtype=torch.float16)), TypeError), (lambda: dict(A=_t(E + 1, R, DI), B=_t(E + 1, DO, R)), ValueError),
    (lambda: dict(y=torch.float16), TypeError), (lambda: dict(y="bf16"), TypeError), (lambda: dict(out=_t(T, DO + 1)), ValueError),
    (lambda: dict(out=_t(T, DO, dtype=torch.float32)), ValueError), (lambda: dict(x=None), TypeError)])
def test_refused(s, kw, error):
    with pytest.raises(error):   # (the tensors are made here: collecting the tests takes no device)
        _planned(s, **kw())
    with pytest.raises(ValueError):
        _planned(s, W=_t(DI, DO).t())   # (not contiguous)
    assert torch.equal(_planned(s), _planned(s))


def test_own_tensors_and_sequences(s):
    y = torch.empty((T, DO), dtype=BF, device="cuda")
    assert _planned(s, out=y) is y
    assert torch.equal(y, _planned(s))
    shared = lambda f, outs=None: moin.moin_lora_linear_planned_shared(s["ctx"], s["plan"], s["x"], f([s["W"]] * 2), f([s["A"]] * 2),
                                                                       f([s["B"]] * 2), 2.0, outs=outs)
    z = [torch.empty_like(y), torch.empty_like(y)]
    ys = shared(list, outs=z)
    assert ys[0] is z[0] and ys[1] is z[1] and isinstance(ys, list)
    assert all(torch.equal(a, b) for a, b in zip(shared(tuple), ys))
    with pytest.raises(ValueError):
        shared(lambda v: v * 3)
    out = (torch.empty(2, dtype=I32, device="cuda"), None, torch.empty(K, dtype=I32, device="cuda"))
    got = moin.moin_route(s["ctx"], s["emb"], s["cent"], want_counts=True, out=out)
    assert got[0] is out[0] and got[1] is None and got[2] is out[2]
    assert int(got[2].sum()) == 2
    for bad in ((None, None), (out[0].long(), None, None), (out[2], None, None)):
        with pytest.raises(ValueError):
            moin.moin_route(s["ctx"], s["emb"], s["cent"], out=bad)
    with pytest.raises(ValueError):
        moin.moin_route_plan(s["ctx"], s["plan"], s["emb"], s["cent"], s["off"], T, E, out=(None, None, None))
    for k in (0, 9):
        with pytest.raises(ValueError):
            moin.moin_route_topk(s["ctx"], s["emb"], s["cent"], k)
    with pytest.raises(TypeError):
        moin.moin_route(s["ctx"], s["emb"].half(), s["cent"].half())
    with pytest.raises(ValueError):
        s["plan"].build(s["off"], s["off"], T, E)
    # lists that nobody else holds
    ys = [moin.moin_lora_linear_planned_shared(s["ctx"], s["plan"], s["x"], (w for w in [s["W"].clone()]), None, None, 2.0)
          for _ in range(3)]
    pygc.collect()
    assert torch.equal(ys[0][0], ys[2][0])


def test_status_and_streams(s):
    with pytest.raises(moin.MoinError) as e:
        _planned(s, x=_t(T, 60), W=_t(DO, 60), A=_t(E, R, 60), B=s["B"])   # d_in % 8
    assert e.value.code < 0 and "moin_lora_linear_planned" in str(e.value)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    y = moin.moin_lora_linear_planned(s["ctx"], s["plan"], s["x"], s["W"], s["A"], s["B"], 2.0, stream=side)
    side.synchronize()
    with torch.cuda.stream(side):
        z = _planned(s)
    side.synchronize()
    assert torch.equal(y, z) and torch.equal(y, _planned(s))
    closed = moin.Plan(s["ctx"]).build(s["off"], s["ids"], T, E)
    closed.close()
    with pytest.raises(moin.MoinError):
        _planned(s, plan=closed)
