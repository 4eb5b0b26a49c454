"""The quantised-base kernel on 128 x 128 tiles: row counts around a tile and a plan tile, widths around a tile's, two
blocks of the contraction and many, every number of parts of a decode-sized product, ranks of one block and several;
against the oracle.  And its bits against the larger tiles'."""
import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from tests import gpu_common as gc
from tests.test_gpu_mx import _case, _mx_check

pytestmark = pytest.mark.gpu

LENS = [300, 256, 1, 130, 511, 128, 129, 255, 127, 40]
IDS = [3, 0, -1, 2, 3, 1, 1, 0, 3, 2]


@pytest.mark.parametrize("d_in,d_out,r,ranks", [(256, 8, 64, None), (256, 136, 64, [64, 8, 56, 0]), (384, 120, 128, None),
                                                (640, 264, 192, [192, 64, 72, 8]), (2048, 128, 64, None)])
def test_prefill_edges(d_in, d_out, r, ranks):
    inp = _case("mx_mid", d_in, d_out, r, 4, LENS, IDS, seed=d_in + d_out)
    _mx_check(inp, f"mx_mid {d_in}->{d_out} r={r}", rank_of_expert=ranks)


@pytest.mark.parametrize("lens,d_out", [([129, 200, 20, 256, 300] * 15, 72), ([20, 400] * 125, 8)])
def test_many_plan_tiles(lens, d_out):   # 90, and more than the 256 whose empty halves are left out
    inp = _case("mx_mid_many", 256, d_out, 64, 4, lens, (np.arange(len(lens)) % 5 - 1).tolist(), seed=d_out)
    _mx_check(inp, f"mx_mid, {len(lens)} sequences, 256->{d_out}")


@pytest.mark.parametrize("T,d_in,d_out", [(1, 256, 136), (17, 768, 8), (127, 1024, 264), (128, 2048, 128), (129, 5632, 72),
                                          (1000, 1280, 520)])
def test_decode_edges(T, d_in, d_out):
    ids = (np.arange(T) * 7 % 6 - 1).tolist()   # -1 .. 4
    inp = _case("mx_mid_decode", d_in, d_out, 64, 5, [1] * T, ids, seed=T + d_in)
    _mx_check(inp, f"mx_mid decode T={T} {d_in}->{d_out}")


@pytest.mark.parametrize("r", [64, 128])
def test_same_bits_as_the_larger_tiles(r):
    inp = _case("mx_mid_bits", 256, 4096, r, 4, [400] * 32, [0, 1, 2, 3] * 8, seed=r)   # 4096 tiles
    Wq, Ws = moin.moin_mx_quantize(gc.ctx(), inp.W, blocked=True)
    call = lambda x, off, e: moin.moin_lora_linear_mx(gc.ctx(), x, off, e, Wq, Ws, inp.A_stack, inp.B_stack, 2.0,
                                                      y_dtype=torch.float32)
    print(f"[gpu] mx, 128 x 128 and 256 x 256 tiles, r={r}", flush=True)
    y = call(inp.x, inp.seq_offsets, inp.expert_ids)
    few = call(inp.x[:1200].contiguous(), inp.seq_offsets[:4].contiguous(), inp.expert_ids[:3].contiguous())   # 384 tiles
    gc.ctx().check()
    assert torch.equal(few, y[:1200])
