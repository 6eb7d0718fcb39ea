"""Performance cases of the error-signature, top-k and injection entry points.

Each case is one call (or the short call sequence of one step) that a user of
the library makes in earnest, from a lone small tensor to a checkpoint, with
inputs shaped like the workloads of the synthetic benchmark.  A case is a dict
of plain values; `prepare` makes its inputs on the GPU from a seed, `run` is
one pass through the public entry points.

Kinds
  one      synchronous signature of one recorded output (Python dict back)
  rfi      random-value corruption of a few positions, then the signature
  topk     synchronous mean of the top 10 % errors of one output
  ckpt     a checkpoint's tensors in one batch: signature, fused injection +
           signature, or top-k mean, stream-ordered
  batch    recorded activations of one layer over a batch of calls: signature,
           or signature followed by the top-k mean fed with its records
  replay   many replayed f16 outputs against one golden
  inject   the injection kernel alone over a list of tensors
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_13544_amd as P

BINS = (-40, 24, 64)
THRESHOLDS = (1e-6, 1e-3)
# a ladder of torch.isclose (atol, rtol) pairs
LADDER = ((1e-8, 1e-5), (1e-5, 1.3e-6), (1e-3, 1.6e-2), (1e-2, 0.0))
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "f64": torch.float64}
SIZE = {"f32": 4, "f16": 2, "bf16": 2, "f64": 8}
REC = P.SIG_BYTES // 8           # 8-byte words of a signature record
TOP = P.TOPK_BYTES // 8          # ... of a top-k record
F32_EXPONENT = 0x7F800000
ODD_ROW = 50257                  # an odd row width (a vocabulary)


def listed():
    return [
        # one recorded f32 layer output, signed as it is produced: the benchmark's single-call size
        {"name": "one_f32_1024x1024", "kind": "one", "golden": "f32", "test": "f32", "n": 1 << 20, "data": "noise"},
        # one replayed f16 [4096, 4096] output against its golden, call by call
        {"name": "one_f16_4096x4096", "kind": "one", "golden": "f16", "test": "f16", "n": 1 << 24, "data": "replay"},
        # runtime fault injection into a small output (a classifier head): three random-value positions, then its
        # signature -- the smallest calls, all latency
        {"name": "rfi_f32_10007", "kind": "rfi", "golden": "f32", "n": 10007, "num_pos": 3},
        # the Analyzer's main score of one layer output
        {"name": "topk_f32_1024x1024", "kind": "topk", "golden": "f32", "test": "f32", "n": 1 << 20, "data": "noise"},
        # a GPT-style 1.3B checkpoint pair (292 tensors, small biases among large matrices)
        {"name": "ckpt_gpt", "kind": "ckpt", "shape": "gpt", "layers": 24, "hidden": 2048, "ffn": 8192, "vocab": 50304,
         "op": "signature"},
        # one assessment step on Llama-shaped layers with both Adam moments: bit flips and signatures in one pass
        # (4 of the 32 layers: three states have to fit on the card)
        {"name": "step_llama_adam", "kind": "ckpt", "shape": "llama", "layers": 4, "hidden": 4096, "ffn": 11008,
         "vocab": 0, "op": "fused"},
        # the top-10 % means of the same kind of checkpoint
        {"name": "topk_llama_adam", "kind": "ckpt", "shape": "llama", "layers": 2, "hidden": 4096, "ffn": 11008,
         "vocab": 0, "op": "topk"},
        # 200 replayed f16 outputs of one op, every tenth with injected flips
        {"name": "replay_f16", "kind": "replay", "calls": 200, "n": 1 << 24},
        # rectified f32 activations [8, 512, 4096] of a convolution or MLP (half the golden zeros): the score step,
        # signature then top-k from its records
        {"name": "score_relu_f32", "kind": "batch", "golden": "f32", "test": "f32", "data": "relu", "pairs": 16,
         "n": 8 * 512 * 4096, "row": 0, "thresholds": "two", "op": "score"},
        # precision comparison: FP32 golden outputs against the same op in FP16
        {"name": "mixed_f32_f16", "kind": "batch", "golden": "f32", "test": "f16", "data": "round", "pairs": 32,
         "n": 4096 * 4096, "row": 0, "thresholds": "two", "op": "signature"},
        # bf16 logits, one contiguous slice per sequence: an odd row width leaves most slices unaligned; a ladder of
        # closeness tests
        {"name": "logits_bf16_odd", "kind": "batch", "golden": "bf16", "test": "bf16", "data": "noise", "pairs": 16,
         "n": 127 * ODD_ROW, "row": ODD_ROW, "thresholds": "ladder", "op": "signature"},
        # injection alone into a list of weights: bit flips, random values, NaN
        {"name": "inject_mixed_models", "kind": "inject", "tensors": 24, "n": 4096 * 4096, "golden": "f32",
         "rate": 1e-6},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["one", "one", "rfi", "topk", "ckpt", "ckpt", "batch", "batch", "replay", "inject"])
    if kind in ("one", "topk"):
        g, t = rng.choice([("f32", "f32"), ("f32", "f32"), ("f16", "f16"), ("bf16", "bf16"), ("f32", "f16"),
                           ("f32", "f64")])
        if kind == "topk" and g != t:
            t = g
        return {"kind": kind, "golden": g, "test": t, "n": _log(rng, 1 << 10, 1 << 25),
                "data": rng.choice(["noise", "relu"] if g == t else ["round"])}
    if kind == "rfi":
        return {"kind": kind, "golden": rng.choice(["f32", "f16", "bf16"]), "n": _log(rng, 1 << 10, 1 << 22),
                "num_pos": rng.choice([1, 3, 5])}
    if kind == "ckpt":
        shape = rng.choice(["gpt", "llama"])
        hidden = 64 * rng.randint(8, 40) + rng.choice([0, 0, 0, 1, 2, 37])
        return {"kind": kind, "shape": shape, "layers": rng.randint(1, 8 if shape == "llama" else 24), "hidden": hidden,
                "ffn": 4 * hidden if shape == "gpt" else (8 * hidden) // 3, "vocab": rng.choice([0, 32000, ODD_ROW]),
                "op": rng.choice(["signature", "fused", "topk"])}
    if kind == "batch":
        g, t = rng.choice([("f32", "f32"), ("f32", "f32"), ("bf16", "bf16"), ("f16", "f16"), ("f32", "f16"),
                           ("f32", "bf16"), ("f32", "f64")])
        row = rng.choice([0, 0, ODD_ROW if g == t else 0])
        n = _log(rng, 1 << 14, 1 << 24)
        if row:
            n = max(1, n // row) * row
        pairs = max(1, min(_log(rng, 4, 256), (1 << 29) // n))
        return {"kind": kind, "golden": g, "test": t, "pairs": pairs, "n": n, "row": row,
                "data": rng.choice(["noise", "relu", "round"]) if g == t == "f32" else
                        (rng.choice(["noise", "relu"]) if g == t else "round"),
                "thresholds": rng.choice(["two", "two", "ladder"]), "op": rng.choice(["signature", "score"])}
    if kind == "replay":
        n = _log(rng, 1 << 18, 1 << 24)
        return {"kind": kind, "calls": max(10, min(_log(rng, 10, 400), (1 << 31) // n)), "n": n}
    n = _log(rng, 1 << 14, 1 << 26)
    return {"kind": kind, "tensors": max(1, min(_log(rng, 1, 64), (1 << 29) // n)), "n": n,
            "golden": rng.choice(["f32", "f16", "bf16"]), "rate": 10.0 ** -rng.randint(4, 9)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed & (2 ** 63 - 1))
    return g


def _randn(n, gen):
    return torch.randn(n, generator=gen, device="cuda", dtype=torch.float32)


def _sparse(n, rate, seed):
    """Positions chosen at a rate, as a device index tensor."""
    rng = np.random.default_rng(seed)
    k = int(rng.binomial(n, rate))
    return torch.from_numpy(rng.integers(0, n, k)).cuda()


def _pair(golden, test, n, data, gen, seed, scale=1.0):
    """One golden/test pair.  noise: the test kernel's relative rounding noise
    around 1e-6 (coarser types round it to a few last-place differences).
    relu: the same under a rectifier, half of the golden values zero.  round:
    the golden rounded to the narrower type (widened back where both sides
    are f32), with 0.1 % outliers.  replay: the golden with a few flipped bits."""
    X = _randn(n, gen) * scale
    if data == "noise":
        rel = 1e-6 if golden == "f32" else 2e-3 if golden == "bf16" else 3e-4
        return X.to(DTYPES[golden]), (X * (1.0 + rel * _randn(n, gen))).to(DTYPES[test])
    if data == "relu":
        eps = 1e-6 if golden == "f32" else 2e-3 if golden == "bf16" else 3e-4
        T = (X + eps * _randn(n, gen)).clamp_min_(0.0).to(DTYPES[test])
        return X.clamp_min_(0.0).to(DTYPES[golden]), T
    if data == "round":
        X = torch.where(torch.rand(n, generator=gen, device="cuda") < 1e-3, X * 100.0, X)
        if test == "f64":
            return X, X.double() * (1.0 + 2.0 ** -24 * _randn(n, gen).double())
        return X.to(DTYPES[golden]), X.to(torch.bfloat16 if test == "f32" else DTYPES[test]).to(DTYPES[test])
    G = X.to(DTYPES[golden])
    T = G.clone()
    pos = _sparse(n, 1e-7 + 4.0 / n, seed)
    bits = torch.int16 if SIZE[golden] == 2 else torch.int32
    T.view(bits)[pos] ^= 1 << 9
    return G, T


def _ckpt_sizes(case):
    h, f, v = case["hidden"], case["ffn"], case["vocab"]
    out = [v * h] if v else []
    for _ in range(case["layers"]):
        if case["shape"] == "gpt":
            out += [h, h, 3 * h * h, 3 * h, h * h, h, h, h, f * h, f, h * f, h]
        else:
            out += [h * h] * 4 + [f * h] * 3 + [h, h]
    return (out + [h, h]) if case["shape"] == "gpt" else out + [h]


def _flat(sizes, align=32):
    """Offsets of the tensors of a padded flat buffer (align elements), and its length."""
    off, pos = [], 0
    for n in sizes:
        off.append(pos)
        pos += -(-n // align) * align
    return off, pos


def _records(d_out, count):
    """The fields of device signature records, by kind (views)."""
    i, f = d_out.view(torch.int64).view(count, REC), d_out.view(torch.float64).view(count, REC)
    return {"counts": i[:, :85], "max_abs": f[:, 85], "index": i[:, 86:90], "max_rel": f[:, 90], "argmax_rel": i[:, 91],
            "sums": f[:, 92:98]}


def _topk_records(d_out, count):
    i, f = d_out.view(torch.int64).view(count, TOP), d_out.view(torch.float64).view(count, TOP)
    return {"counts": i[:, :3], "values": f[:, 3:]}


def _buffer(words, count):
    return torch.zeros(words * 8 * count, dtype=torch.uint8, device="cuda")


def _tensors(case, seed):
    """The (golden, test) pairs of a case and the flat buffers they live in (checkpoints)."""
    gen = _gen(seed)
    kind = case["kind"]
    if kind in ("one", "topk"):
        return [_pair(case["golden"], case["test"], case["n"], case["data"], gen, seed)], []
    if kind == "rfi":
        G, T = _pair(case["golden"], case["golden"], case["n"], "noise", gen, seed)
        return [(G, T)], []
    if kind == "ckpt":
        sizes = _ckpt_sizes(case)
        off, total = _flat(sizes)
        states = [0.02] if case["shape"] == "gpt" else [0.02, 1e-3, 1e-6]     # weights (Adam m, Adam v)
        pairs, flats = [], []
        for s, scale in enumerate(states):
            G, T = torch.zeros(total, device="cuda"), torch.zeros(total, device="cuda")
            step = 1 << 28
            for a in range(0, total, step):
                b = min(total, a + step)
                X = _randn(b - a, gen)
                if s == 2:
                    X.mul_(X)
                X.mul_(scale)
                G[a:b] = X
                T[a:b] = (X.double() * (1.0 + (1e-6 if case["shape"] == "gpt" else 1e-7)
                                        * _randn(b - a, gen).double())).float()
            T[_sparse(total, 1e-9, seed + s)] = float("nan")
            pairs += [(G[o:o + n], T[o:o + n]) for o, n in zip(off, sizes)]
            flats.append(T)
        return pairs, flats
    if kind == "batch":
        n, count = case["n"], case["pairs"]
        if case["row"]:
            # slices of one logits tensor: sequence k starts wherever its rows start
            G, T = _pair(case["golden"], case["test"], n * count, case["data"], gen, seed)
            return [(G[k * n:(k + 1) * n], T[k * n:(k + 1) * n]) for k in range(count)], []
        return [_pair(case["golden"], case["test"], n, case["data"], gen, seed + k) for k in range(count)], []
    if kind == "replay":
        n = case["n"]
        G = _randn(n, gen).half()
        pairs = []
        for k in range(case["calls"]):
            T = G.clone()
            if k % 10 == 9:
                pos = _sparse(n, 1e-7 + 1.0 / n, seed + k)
                T.view(torch.int16)[pos] ^= 1 << (k % 15)
            pairs.append((G, T))
        return pairs, []
    raise ValueError(kind)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "inject":
        gen = _gen(seed)
        ts = [_randn(case["n"], gen).to(DTYPES[case["golden"]]) for _ in range(case["tensors"])]
        mask = F32_EXPONENT if case["golden"] == "f32" else 0x7FFF
        models = [P.MODEL_BITFLIP, P.MODEL_BITFLIP, P.MODEL_VALUE, P.MODEL_NAN]
        items = P.PreparedItems([(t, seed * 64 + k, case["rate"], mask, models[k % 4]) for k, t in enumerate(ts)])
        return {"kind": kind, "items": items, "tensors": ts,
                "counts": torch.zeros(len(ts), dtype=torch.int64, device="cuda")}
    pairs, flats = _tensors(case, seed)
    state = {"kind": kind, "pairs": pairs, "seed": seed, "flats": flats, "op": case.get("op", "signature"),
             "num_pos": case.get("num_pos", 0),
             "mixed": case.get("golden") != case.get("test", case.get("golden")),
             "thresholds": LADDER if case.get("thresholds") == "ladder" else THRESHOLDS}
    if kind in ("one", "rfi", "topk"):
        return state
    count = len(pairs)
    if not state["mixed"]:
        state["plan"] = P.PreparedPairs(pairs)
    state["out"] = _buffer(REC, count)
    state["fields"] = _records(state["out"], count)
    if state["op"] in ("topk", "score"):
        state["top"] = _buffer(TOP, count)
        state["top_fields"] = _topk_records(state["top"], count)
    if state["op"] == "fused":
        state["seeds"] = [seed * 1000 + k for k in range(count)]
        state["flips"] = torch.zeros(count, dtype=torch.int64, device="cuda")
        # a NaN or infinite value compares by its bits
        state["flat_bits"] = [t.view(torch.int32) for t in flats]
    return state


def run(state):
    kind, op, pairs = state["kind"], state.get("op"), state.get("pairs")
    if kind == "one":
        G, T = pairs[0]
        d = P.signature_mixed(G, T, BINS, THRESHOLDS) if state["mixed"] else P.signature(G, T, BINS, THRESHOLDS)
        d["hist"] = np.array(d["hist"])
        return d
    if kind == "rfi":
        G, T = pairs[0]
        pos = P.corrupt_positions(T, state["seed"], P.MODEL_VALUE, state["num_pos"])
        d = P.signature(G, T, BINS, THRESHOLDS)
        d["hist"] = np.array(d["hist"])
        return [np.array(pos), d]
    if kind == "topk":
        return P.topk_mean(*pairs[0])
    if kind == "inject":
        P.inject_batched_async(state["items"], state["counts"])
        return [state["counts"]] + [t.view(torch.int16 if t.element_size() == 2 else torch.int32)
                                    for t in state["tensors"][:60]]
    if op == "fused":
        P.inject_signature_batched_async(state["plan"], state["seeds"], 1e-8, F32_EXPONENT, state["out"], state["flips"],
                                         BINS, THRESHOLDS)
        return [state["fields"], state["flips"]] + state["flat_bits"]
    if op == "topk":
        P.topk_mean_batched_async(state["plan"], state["top"])
        return state["top_fields"]
    if state["mixed"]:
        P.signature_mixed_batched_async(pairs, state["out"], BINS, state["thresholds"])
        if op == "score":
            P.topk_mean_mixed_from_signature_batched_async(pairs, state["out"], state["top"], BINS)
            return [state["fields"], state["top_fields"]]
        return state["fields"]
    P.signature_batched_async(state["plan"], state["out"], BINS, state["thresholds"])
    if op == "score":
        P.topk_mean_from_signature_batched_async(state["plan"], state["out"], state["top"], BINS)
        return [state["fields"], state["top_fields"]]
    return state["fields"]


# ---------------------------------------------------------------------------
# work, tolerance, 64-bit values
# ---------------------------------------------------------------------------
def work(case):
    """Bytes: golden and test read once (a shared golden once), records written.
    A signature's binary64 arithmetic is about 10 operations per element; the
    injection draws are integer operations (about 10 per element) that touch
    memory only at chosen elements -- a random-value item needs no more than
    its chosen elements either."""
    kind = case["kind"]
    if kind == "inject":
        n = case["n"] * case["tensors"]
        return {"bytes": max(64.0, n * min(1.0, case["rate"]) * 64), "flops": 10.0 * n}
    if kind == "ckpt":
        n = sum(_ckpt_sizes(case)) * (1 if case["shape"] == "gpt" else 3)
        count = len(_ckpt_sizes(case)) * (1 if case["shape"] == "gpt" else 3)
        return {"bytes": 8.0 * n + P.SIG_BYTES * count, "flops": (20.0 if case["op"] == "fused" else 10.0) * n}
    if kind == "replay":
        return {"bytes": 2.0 * case["n"] * (case["calls"] + 1) + P.SIG_BYTES * case["calls"],
                "flops": 10.0 * case["n"] * case["calls"]}
    n, count = case["n"], case.get("pairs", 1)
    b = n * (SIZE[case["golden"]] + SIZE[case.get("test", case["golden"])])
    # the score step's two calls each stream the tensors; one stream would do
    return {"bytes": float(count) * (b + P.SIG_BYTES), "flops": 10.0 * n * count}


def tolerance(case):
    """Counts, indices, maxima, positions and tensor bits are exact; the
    binary64 sums may be taken in any order.  The path differs from sums of
    another order by at most about 1e-15, and a relative-error term may carry
    another 2^-47 from its reciprocal: 1e-13 covers both with room."""
    if case["kind"] == "inject":
        return "exact"
    return {"rel": 1e-13, "max": 1e-13, "differ": 0.0}


def _sums64(G, T):
    """max_abs, max_rel and the six sums of one pair, in binary64."""
    part, ma, mr = torch.zeros(6, dtype=torch.float64, device="cuda"), [], []
    for a in range(0, G.numel(), 1 << 25):
        g, t = G[a:a + (1 << 25)].double(), T[a:a + (1 << 25)].double()
        e = torch.where(g == t, 0.0, (t - g).abs())
        valid = ~(g.isnan() | t.isnan())
        ma.append(torch.where(valid, e, -1.0).max())
        fin = g.isfinite() & t.isfinite()
        g, t, e = torch.where(fin, g, 0.0), torch.where(fin, t, 0.0), torch.where(fin, e, 0.0)
        r = torch.where(g != 0, e / torch.where(g != 0, g.abs(), 1.0), 0.0)
        mr.append(torch.where(fin & (g != 0), r, -1.0).max())
        part += torch.stack([e.sum(), (e * e).sum(), r.sum(), (g * g).sum(), (t * t).sum(), (g * t).sum()])
    neg = lambda v: torch.where(v < 0, float("nan"), v)  # noqa: E731
    return neg(torch.stack(ma).max()), neg(torch.stack(mr).max()), part


def _topk64(G, T):
    """kth value, sum and mean of the ceil(n_valid / 10) largest errors."""
    g, t = G.double(), T.double()
    e = torch.where(g == t, 0.0, (t - g).abs())[~(g.isnan() | t.isnan())]
    k = -(-e.numel() // 10)
    top = torch.sort(e, descending=True).values[:k]
    s = top.sum()
    return torch.stack([top[-1], s, s / k])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("inject", "rfi") or case.get("op") == "fused":
        return None                  # the flips themselves are whole values, compared exactly
    if work(case)["bytes"] > 14e9:
        return None
    pairs, _ = _tensors(case, seed)
    if kind == "topk":
        kth, s, m = (float(x) for x in _topk64(*pairs[0]))
        return {"kth_value": kth, "sum_topk": s, "mean_topk": m}
    if kind == "one":
        ma, mr, s = _sums64(*pairs[0])
        names = ("sum_abs", "sum_sq", "sum_rel", "sum_g2", "sum_t2", "sum_gt")
        return {"max_abs": float(ma), "max_rel": float(mr), **{k: float(v) for k, v in zip(names, s)}}
    top = {"counts": None, "values": torch.stack([_topk64(*p) for p in pairs])} \
        if case.get("op") in ("topk", "score") else None
    if case.get("op") == "topk":
        return top
    rows = [_sums64(*p) for p in pairs]
    sig = {"counts": None, "max_abs": torch.stack([r[0] for r in rows]), "index": None,
           "max_rel": torch.stack([r[1] for r in rows]), "argmax_rel": None, "sums": torch.stack([r[2] for r in rows])}
    return [sig, top] if top else sig
