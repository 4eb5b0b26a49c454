"""The prefill kernel on 64 x 64 tiles, for calls of few tiles: rows around a quarter of a plan tile, widths and contractions
on both sides of a block, up to the plan tiles it takes; against torch in fp64, its bits against the 128 x 128 tiles', and
those (which take the same batch four times over) at the same edges.  Its assembly as that of the larger tiles."""
import re

import numpy as np
import pytest
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl
from tests import gpu_common as gc
from tests.test_asm_mfma_hazards import MIN_GAP, _device_asm, _regs, _whole_bodies
from tests.test_gpu_decode_stream import _check
from tests.test_gpu_prefill_mid import E, IDS, LENS, _run


@pytest.mark.gpu
@pytest.mark.parametrize("times", [1, 4])
@pytest.mark.parametrize("d_in,d_out,r,ranked,f32", [
    (8, 8, 8, False, True), (64, 64, 64, True, True), (72, 72, 136, False, False), (192, 56, 24, True, False), (520, 264, 40, True, True),
    (1000, 200, 32, False, True), (2048, 256, 128, True, False)])
def test_edges(times, d_in, d_out, r, ranked, f32):
    y, ref = _run(LENS * times, np.tile(IDS, times), d_in, d_out, r, ranked, f32)
    if f32:
        _check(y, ref, d_in, r)
    else:   # rounded to bf16: half a unit of the last of 8 bits
        assert bool(((y.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all())


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[64, 65, 63, 128, 129, 1, 192, 193, 255, 256, 257], [30] * 3 + [1500], [100] * 28 + [3000]])
@pytest.mark.parametrize("d_in,r", [(192, 64), (200, 24)])
def test_same_bits_in_a_larger_batch(lens, d_in, r):
    d_out, S = 136, len(lens)
    more = lens + [400] * 60
    ids = np.tile(np.array([0, -1, 1, 2, 3], dtype=np.int32), len(more))[:len(more)]
    w = wl.LinearWorkload("fine", d_in, d_out, r, E, more, "uniform", scale=2.0, seed=d_in + S)
    inp = wl.make_linear_inputs(w, "cuda", expert_ids=ids)
    inp.A_stack[4] = float("nan")   # (no sequence uses it)
    inp.B_stack[4] = float("inf")
    T = sum(lens)
    assert T > 1024
    print(f"[gpu] prefill on 64 x 64 tiles, {S} sequences of {T} tokens, {d_in}->{d_out} r={r}", flush=True)
    call = lambda x, off, e: moin.moin_lora_linear(gc.ctx(), x, off, e, inp.W, inp.A_stack, inp.B_stack, 2.0, y_dtype=torch.float32)
    few = call(inp.x[:T].contiguous(), inp.seq_offsets[:S + 1].contiguous(), inp.expert_ids[:S].contiguous())
    all_ = call(inp.x, inp.seq_offsets, inp.expert_ids)
    gc.ctx().check()
    assert bool(torch.isfinite(all_).all()) and torch.equal(few, all_[:T])


def test_assembly():
    bodies = _whole_bodies(_device_asm("linear_mid.hip"), "linear_fine_kernel")
    assert len(bodies) == 4
    for sym, lines in bodies:
        assert not any(re.search(r"\bscratch_(load|store)", l) for l in lines), f"{sym} spills to scratch"
        in_asm, count, n_mfma, last = False, 0, 0, {}
        for t in (l.strip() for l in lines):
            in_asm = (in_asm or t.startswith(";;#ASMSTART")) and not t.startswith(";;#ASMEND")
            if not t or t[0] in ";." or t.endswith(":"):
                continue
            op, _, rest = t.partition(" ")
            args = [a.strip() for a in rest.split(",")]
            count += (int(args[0]) + 4) // 4 if op == "s_nop" else 1
            if op.startswith("v_mfma"):
                n_mfma += 1
                last.update({r: count for r in _regs(args[0])})
            elif op.startswith("v_accvgpr") and not in_asm:
                for r in set().union(*(_regs(a) for a in args)):
                    assert count - last.get(r, -10 ** 9) > MIN_GAP, f"{sym}: `{t}`"
        assert n_mfma >= 32, f"{sym}: {n_mfma} MFMAs"
