"""The work that a server of topic-routed adapters has libmoin do, as cases that can be timed.

``listed()`` names twelve, ``draw()`` gives more of the same ranges.  A case is a dict of plain values; its
``kind`` says which calls one pass makes:

* ``step``    routing of a batch of requests, grouping, and one projection (what a new request starts with);
* ``layer``   the seven projections of one transformer layer on a batch that is already routed: prefill
              (long sequences) or decode (one token per sequence), on a bf16 or an MXFP8 base;
* ``tokens``  one projection of a batch of very short sequences, down to one expert per token;
* ``route``   assignment of a set of embeddings to topics, with the histogram;
* ``topk``    the nearest topics of every query, and merged adapters for the first few;
* ``kmeans``  Lloyd iterations on a table of embeddings.

Inputs are seeded and synthetic: activations N(0,1), weights and adapters N(0, 1/fan_in), unit-length
embeddings scattered around topics that are drawn unevenly, expert use by a Zipf law.
"""
import math

import numpy as np
import torch

from paper_2410_09687_amd import moin
from paper_2410_09687_amd import workloads as wl

BF16, F32 = torch.bfloat16, torch.float32

# d_in -> d_out of a layer's projections (2048-wide model, grouped k / v heads)
QKV, O, GATE_UP, DOWN = (2048, 256, 256), 2048, (5632, 5632), 2048
D_MODEL, D_FF = 2048, 5632


# ---- the cases ------------------------------------------------------------------------------------------

def listed():
    return [
        # Four short requests against a toy model: the smallest call there is, all latency.
        dict(name="step_tiny", kind="step", S=4, len_lo=64, len_hi=64, d_in=256, d_out=256, r=16, E=8, K=8, D=256,
             emb="f32", y="f32", act="", ranked=False, planned=False),
        # A full prefill batch of 64 requests of 512 tokens through one attention projection.
        dict(name="step_prefill", kind="step", S=64, len_lo=512, len_hi=512, d_in=2048, d_out=2048, r=64, E=500,
             K=500, D=768, emb="bf16", y="bf16", act="", ranked=False, planned=True),
        # A handful of requests of uneven length on rank-16 adapters, some of smaller rank: what a lightly
        # loaded server prefills; embeddings as the embedder gives them, in fp32.
        dict(name="step_ragged", kind="step", S=7, len_lo=40, len_hi=900, d_in=2048, d_out=5632, r=16, E=470, K=500,
             D=384, emb="f32", y="bf16", act="silu", ranked=True, planned=True),
        # A large prefill: 32 sequences of 2048 tokens through a whole layer, rank-128 adapters.
        dict(name="layer_prefill", kind="layer", S=32, len_lo=2048, len_hi=2048, r=128, E=500, zipf=1.5, mx=False),
        # The same layer on an MXFP8 base, sequences of uneven length.
        dict(name="layer_prefill_mx", kind="layer", S=24, len_lo=100, len_hi=1900, r=64, E=500, zipf=1.1, mx=True),
        # Decode with few users and with many: one token per sequence, hundreds of distinct adapters.
        dict(name="layer_decode_8", kind="layer", S=8, len_lo=1, len_hi=1, r=128, E=2000, zipf=1.1, mx=False),
        dict(name="layer_decode_256", kind="layer", S=256, len_lo=1, len_hi=1, r=128, E=2000, zipf=1.1, mx=False),
        # One expert per token.
        dict(name="tokens_8192", kind="tokens", S=8192, len_lo=1, len_hi=1, d_in=2048, d_out=5632, r=128, E=5000,
             zipf=1.1),
        # Requests routed as they arrive, on fp32 embeddings, topics without an adapter left out.
        dict(name="route_requests", kind="route", N=1000, K=5000, D=384, emb="f32", retained=True),
        # A million documents assigned to 5000 topics.
        dict(name="route_bulk", kind="route", N=1 << 20, K=5000, D=768, emb="bf16", retained=False),
        # Nearest topics of a batch of queries, merged adapters for the first four.
        dict(name="topk_merge", kind="topk", N=1000, K=5000, D=768, emb="bf16", k=4, merges=4, r=32, E=500),
        # Three Lloyd iterations (and the final assignment) on a quarter of a million documents.
        dict(name="kmeans_fit", kind="kmeans", N=1 << 18, K=5000, D=768, emb="bf16", iters=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "layer", "layer", "layer", "tokens", "route", "route", "topk", "kmeans"])
    if kind == "step":
        d_in, d_out = rng.choice([(256, 256), (2048, 2048), (2048, 256), (2048, 5632), (5632, 2048), (1024, 1416),
                                  (2048, 2000), (1000, 2048)])
        S = _log(rng, 1, 64)
        hi = _log(rng, 16, 1024)
        return dict(kind=kind, S=S, len_lo=max(1, hi // rng.choice([1, 2, 20])), len_hi=hi, d_in=d_in, d_out=d_out,
                    r=8 * rng.choice([1, 2, 4, 4, 5, 8, 8, 16]), E=_log(rng, 8, 480), K=500, D=rng.choice([256, 384, 768]),
                    emb=rng.choice(["f32", "bf16", "bf16"]), y=rng.choice(["bf16", "bf16", "f32"]),
                    act=rng.choice(["", "", "silu"]), ranked=rng.random() < 0.3, planned=rng.random() < 0.7)
    if kind == "layer":
        mx = rng.random() < 0.35
        r = rng.choice([64, 128]) if mx else rng.choice([16, 32, 64, 128, 128])
        if rng.random() < 0.5:
            return dict(kind=kind, S=_log(rng, 1, 1024), len_lo=1, len_hi=1, r=r, E=_log(rng, 50, 2000), zipf=1.1, mx=mx)
        S, hi = _log(rng, 1, 32), _log(rng, 64, 2048)
        return dict(kind=kind, S=S, len_lo=max(1, hi // rng.choice([1, 2, 20])), len_hi=hi, r=r, E=500,
                    zipf=rng.choice([1.1, 1.5]), mx=mx)
    if kind == "tokens":
        d_in, d_out = rng.choice([(2048, 5632), (5632, 2048), (2048, 2048)])
        hi = rng.choice([1, 1, 4, 24])
        return dict(kind=kind, S=_log(rng, 1100, 8192) // (1 if hi == 1 else hi // 2 + 1) + 1, len_lo=1, len_hi=hi,
                    d_in=d_in, d_out=d_out, r=rng.choice([32, 64, 128]), E=_log(rng, 50, 3000), zipf=1.1)
    if kind == "route":
        emb = rng.choice(["f32", "bf16", "bf16"])
        return dict(kind=kind, N=_log(rng, 1, 16384 if emb == "f32" else 1 << 20), K=_log(rng, 16, 5000),
                    D=rng.choice([64, 200, 256, 384, 768]), emb=emb, retained=rng.random() < 0.4)
    if kind == "topk":
        return dict(kind=kind, N=_log(rng, 1, 4096), K=_log(rng, 16, 5000), D=rng.choice([64, 200, 384, 768]),
                    emb=rng.choice(["f32", "bf16"]), k=rng.randint(1, 8), merges=rng.randint(0, 4),
                    r=8 * rng.choice([1, 2, 4]), E=_log(rng, 16, 500))
    emb = rng.choice(["bf16", "bf16", "f32"])
    return dict(kind=kind, N=_log(rng, 1000, 8192 if emb == "f32" else 1 << 18), K=_log(rng, 16, 5000),
                D=rng.choice([64, 200, 384, 768]), emb=emb, iters=rng.randint(1, 3))


# ---- inputs ---------------------------------------------------------------------------------------------

def _lens(c):
    """Sequence lengths: a property of the case, the same for every seed."""
    rng = np.random.default_rng(c["S"] * 1009 + c["len_lo"] * 31 + c["len_hi"])
    return rng.integers(c["len_lo"], c["len_hi"] + 1, size=c["S"]).tolist()


def _normal(g, shape, std=1.0, dtype=BF16):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)


def _stacks(g, E, r, d_in, d_out):
    return _normal(g, (E, r, d_in), d_in ** -0.5), _normal(g, (E, d_out, r), r ** -0.5)


def _unit(v, dtype):
    return (v / v.norm(dim=1, keepdim=True)).to(dtype)


def _topics(g, seed, N, K, D, dtype):
    """K unit topic vectors and N unit embeddings scattered around them, topics drawn by a Zipf law."""
    cent = _normal(g, (K, D), 1.0, F32)
    which = torch.from_numpy(wl.draw_expert_ids(N, K, "zipf", 0.7, seed * 17 + 3).astype(np.int64)).cuda()
    emb = torch.empty((N, D), dtype=dtype, device="cuda")
    for lo in range(0, N, 1 << 17):
        hi = min(N, lo + (1 << 17))
        emb[lo:hi] = _unit(cent[which[lo:hi]] * 0.6 + _normal(g, (hi - lo, D), 1.0, F32), dtype)
    return emb, _unit(cent, dtype)


def _slots(K, E, seed):
    """slot_of_centroid: min(K, E) of the topics have an adapter, the others none."""
    return torch.from_numpy(wl.retained_slot_table(K, min(K, E), seed * 13 + 7)).cuda()


def _offsets(lens):
    return torch.from_numpy(wl.seq_offsets_of(lens)).cuda()


def _ids(c, S, seed):
    return torch.from_numpy(wl.draw_expert_ids(S, c["E"], "zipf", c["zipf"], seed * 7 + 1, perm_seed=seed)).cuda()


def _ranks(c, seed):
    """Each adapter's own rank: full for a third of them, less for the others, always a multiple of 8."""
    rng = np.random.default_rng(seed * 3 + 2)
    r8 = c["r"] // 8
    share = rng.choice([1.0, 0.5, 0.25], size=c["E"])
    return torch.from_numpy((8 * np.maximum(1, (share * r8).astype(np.int64))).astype(np.int32)).cuda()


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 11)
    ctx = moin.Context(torch.cuda.current_device())
    st = dict(case=c, ctx=ctx)
    kind = c["kind"]
    if kind == "step":
        if c["act"]:
            ctx.set_adapter_activation(c["act"])
        lens = _lens(c)
        st["T"] = sum(lens)
        st["off"] = _offsets(lens)
        dt = F32 if c["emb"] == "f32" else BF16
        st["emb"], st["cent"] = _topics(g, seed, c["S"], c["K"], c["D"], dt)
        st["slot"] = _slots(c["K"], c["E"], seed)
        st["ranks"] = _ranks(c, seed) if c["ranked"] else None
        st["x"] = _normal(g, (st["T"], c["d_in"]))
        st["W"] = _normal(g, (c["d_out"], c["d_in"]), c["d_in"] ** -0.5)
        st["A"], st["B"] = _stacks(g, c["E"], c["r"], c["d_in"], c["d_out"])
        st["y"] = F32 if c["y"] == "f32" else BF16
        st["plan"] = moin.Plan(ctx) if c["planned"] else None
    elif kind == "layer":
        lens = _lens(c)
        T = st["T"] = sum(lens)
        st["off"], st["ids"], st["plan"] = _offsets(lens), _ids(c, c["S"], seed), moin.Plan(ctx)
        st["h"] = _normal(g, (T, D_MODEL))
        for name, d_in, d_outs in (("qkv", D_MODEL, QKV), ("o", D_MODEL, (O,)), ("gu", D_MODEL, GATE_UP),
                                   ("down", D_FF, (DOWN,))):
            W = [_normal(g, (d, d_in), d_in ** -0.5) for d in d_outs]
            if c["mx"]:   # the base is quantised once, when the model is loaded
                W = [moin.moin_mx_quantize(ctx, w, blocked=True) for w in W]
            AB = [_stacks(g, c["E"], c["r"], d_in, d) for d in d_outs]
            st[name] = (W, [a for a, _ in AB], [b for _, b in AB])
        if c["mx"]:
            st["codes"] = [(torch.empty((T, D_MODEL), dtype=torch.uint8, device="cuda"),
                            torch.empty((D_MODEL // 128, T, 4), dtype=torch.uint8, device="cuda")) for _ in range(2)]
    elif kind == "tokens":
        lens = _lens(c)
        st["T"] = sum(lens)
        st["off"], st["ids"], st["plan"] = _offsets(lens), _ids(c, c["S"], seed), moin.Plan(ctx)
        st["x"] = _normal(g, (st["T"], c["d_in"]))
        st["W"] = _normal(g, (c["d_out"], c["d_in"]), c["d_in"] ** -0.5)
        st["A"], st["B"] = _stacks(g, c["E"], c["r"], c["d_in"], c["d_out"])
    elif kind == "route":
        st["emb"], st["cent"] = _topics(g, seed, c["N"], c["K"], c["D"], F32 if c["emb"] == "f32" else BF16)
        st["slot"] = _slots(c["K"], max(1, c["K"] * 47 // 50), seed) if c["retained"] else None
    elif kind == "topk":
        st["emb"], st["cent"] = _topics(g, seed, c["N"], c["K"], c["D"], F32 if c["emb"] == "f32" else BF16)
        st["slot"] = _slots(c["K"], c["E"], seed)
        st["A"], st["B"] = _stacks(g, c["E"], c["r"], D_MODEL, D_FF)
        m, R = min(c["merges"], c["N"]), c["k"] * c["r"]
        st["A_out"] = torch.empty((m, R, D_MODEL), dtype=BF16, device="cuda")
        st["B_out"] = torch.empty((m, D_FF, R), dtype=BF16, device="cuda")
    elif kind == "kmeans":
        st["emb"], _ = _topics(g, seed, c["N"], max(8, c["K"] // 2), c["D"], F32 if c["emb"] == "f32" else BF16)
        pick = np.random.default_rng(seed * 5 + 4).choice(c["N"], size=c["K"], replace=c["K"] > c["N"])
        st["first"] = st["emb"][torch.from_numpy(pick).cuda()].contiguous()
        st["cent"] = torch.empty_like(st["first"])
    else:
        raise ValueError("unknown kind of case: %r" % kind)
    return st


# ---- one pass -------------------------------------------------------------------------------------------

def _run_step(st):
    ctx, c = st["ctx"], st["case"]
    if st["plan"] is None:
        eids, cids, counts = moin.moin_route(ctx, st["emb"], st["cent"], st["slot"], want_counts=True)
        y = moin.moin_lora_linear(ctx, st["x"], st["off"], eids, st["W"], st["A"], st["B"], 2.0, y_dtype=st["y"],
                                  rank_of_expert=st["ranks"])
    else:
        eids, cids, counts = moin.moin_route_plan(ctx, st["plan"], st["emb"], st["cent"], st["off"], st["T"], c["E"],
                                                  st["slot"], rank_of_expert=st["ranks"], want_centroid_ids=True,
                                                  want_counts=True, same_centroids=True)
        y = moin.moin_lora_linear_planned(ctx, st["plan"], st["x"], st["W"], st["A"], st["B"], 2.0, y_dtype=st["y"])
    return eids, cids, counts, y


def _run_layer(st):
    ctx, plan, c = st["ctx"], st["plan"], st["case"]
    plan.build(st["off"], st["ids"], st["T"], c["E"])

    def one(name, x):
        W, A, B = st[name]
        if c["mx"]:
            return moin.moin_lora_linear_mx_planned(ctx, plan, x, W[0][0], W[0][1], A[0], B[0], 2.0)
        return moin.moin_lora_linear_planned(ctx, plan, x, W[0], A[0], B[0], 2.0)

    def shared(name, x, i):
        W, A, B = st[name]
        if c["mx"]:   # the first projection quantises the input they share
            xq, xs = st["codes"][i]
            return [moin.moin_lora_linear_mx_planned(ctx, plan, x, w[0], w[1], a, b, 2.0, xq=xq, xs=xs, emit=n == 0)
                    for n, (w, a, b) in enumerate(zip(W, A, B))]
        return moin.moin_lora_linear_planned_shared(ctx, plan, x, W, A, B, 2.0)

    q, k, v = shared("qkv", st["h"], 0)
    o = one("o", q)
    gate, up = shared("gu", o, 1)
    down = one("down", gate)
    return dict(q=q, k=k, v=v, o=o, gate=gate, up=up, down=down)


def _run_tokens(st):
    st["plan"].build(st["off"], st["ids"], st["T"], st["case"]["E"])
    return moin.moin_lora_linear_planned(st["ctx"], st["plan"], st["x"], st["W"], st["A"], st["B"], 2.0)


def _run_route(st):
    return moin.moin_route(st["ctx"], st["emb"], st["cent"], st["slot"], retained_only=st["case"]["retained"],
                           want_counts=True)


def _run_topk(st):
    ctx = st["ctx"]
    eids, cids, d2 = moin.moin_route_topk(ctx, st["emb"], st["cent"], st["case"]["k"], st["slot"])
    if st["A_out"].shape[0]:
        weights = torch.softmax(-d2, dim=1)
        for m in range(st["A_out"].shape[0]):
            moin.moin_merge_adapters(ctx, st["A"], st["B"], eids[m], weights[m], st["A_out"][m], st["B_out"][m])
    return eids, cids, d2, st["A_out"], st["B_out"]


def _run_kmeans(st):
    st["cent"].copy_(st["first"])
    ids, counts, inertia = moin.moin_kmeans_fit(st["ctx"], st["emb"], st["cent"], st["case"]["iters"])
    return ids, counts, inertia, st["cent"]


def run(state):
    return {"step": _run_step, "layer": _run_layer, "tokens": _run_tokens, "route": _run_route, "topk": _run_topk,
            "kmeans": _run_kmeans}[state["case"]["kind"]](state)


# ---- what a pass cannot do without ----------------------------------------------------------------------

def _linear_work(T, experts, d_in, d_out, r, w_bytes=2.0, y_bytes=2.0):
    """x, W and every distinct adapter read once, y written once; base, shrink and expand products."""
    return (2.0 * T * d_in + w_bytes * d_in * d_out + 2.0 * experts * r * (d_in + d_out) + y_bytes * T * d_out,
            2.0 * T * d_in * d_out + 2.0 * T * r * (d_in + d_out))


def _distinct(S, E, s):
    """Expected number of distinct experts of S Zipf draws."""
    return float((1.0 - (1.0 - wl.zipf_probabilities(E, s)) ** S).sum())


def work(case):
    c = case
    kind = c["kind"]
    if kind in ("step", "layer", "tokens"):
        T = float(sum(_lens(c)))
    if kind == "step":
        eb = 4.0 if c["emb"] == "f32" else 2.0
        n = min(c["S"], c["E"])
        b, f = _linear_work(T, n, c["d_in"], c["d_out"], c["r"] * (0.58 if c["ranked"] else 1.0),
                            y_bytes=4.0 if c["y"] == "f32" else 2.0)
        return dict(bytes=b + eb * (c["S"] + c["K"]) * c["D"], flops=f + 2.0 * c["S"] * c["K"] * c["D"])
    if kind == "layer":
        n = _distinct(c["S"], c["E"], c["zipf"])
        wb = 33.0 / 32.0 if c["mx"] else 2.0
        b = f = 0.0
        for d_in, d_outs in ((D_MODEL, QKV), (D_MODEL, (O,)), (D_MODEL, GATE_UP), (D_FF, (DOWN,))):
            for i, d in enumerate(d_outs):
                bi, fi = _linear_work(T, n, d_in, d, c["r"], wb)
                b, f = b + bi - (2.0 * T * d_in if i else 0.0), f + fi
        return dict(bytes=b, flops=f)
    if kind == "tokens":
        b, f = _linear_work(T, _distinct(c["S"], c["E"], c["zipf"]), c["d_in"], c["d_out"], c["r"])
        return dict(bytes=b, flops=f)
    eb = 4.0 if c["emb"] == "f32" else 2.0
    tables, dots = eb * (c["N"] + c["K"]) * c["D"], 2.0 * c["N"] * c["K"] * c["D"]
    if kind == "route":
        return dict(bytes=tables + 8.0 * c["N"] + 4.0 * c["K"], flops=dots)
    if kind == "topk":
        m = min(c["merges"], c["N"])
        return dict(bytes=tables + 12.0 * c["N"] * c["k"] + 4.0 * m * c["k"] * c["r"] * (D_MODEL + D_FF), flops=dots)
    # kmeans: every assignment and every update (or final objective) reads the table
    n = c["iters"] + 1
    return dict(bytes=2.0 * n * tables + 4.0 * c["N"], flops=n * (dots + 3.0 * c["N"] * c["D"]))


def tolerance(case):
    # Against the same passes with sums in fp64: 1.7e-3 (bf16 results) and 2.2e-6 (fp32 results) for the linear
    # layers, 4e-8 for topk's distances, no differing id anywhere; a bf16 merged adapter and a bf16 centre differ
    # where a sum in another order tips a rounding, an id where two distances tie to the last bits.
    kind = case["kind"]
    if kind == "step":
        return dict(rel=1e-5 if case["y"] == "f32" else 7e-3, differ=1e-3)
    if kind in ("layer", "tokens"):
        return dict(rel=7e-3)
    if kind == "route":
        return dict(rel=0.0, differ=1e-3)
    return dict(rel=1e-3, differ=1e-3)
