"""GPU parity where the chunk pass has to look at single elements: zero goldens
(a rectifier's output), elements left to the generic path (one to nearly all
of a vector, so that the list of 64 fills and drains), unaligned tensors and
the ragged rest of a chunk, against the oracle.  Tolerances as in tests/parity.py."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2609_13544_amd as P
import synth
from tests.parity import _SPECIALS, assert_parity, float_to_bits, oracle_sig, records_equal, special_pair, to_device

pytestmark = pytest.mark.gpu

VEC = {0: 4, 1: 8, 2: 8}             # elements per lane vector
LADDER = ((1e-8, 1e-5), (1e-3, 1.6e-2), (1e-2, 0.0))


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    P.lib()
    assert oracle.lib()
    yield
    torch.cuda.synchronize()


def _relu(n, code, seed, eps=0.0):
    """Rectified values, half of them zero; with eps a few tests cross zero."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal(n)
    g = float_to_bits(np.maximum(x, 0.0), code).copy()
    t = float_to_bits(np.maximum(x * (1 + 1e-3 * rng.standard_normal(n)) + eps * rng.standard_normal(n), 0.0), code)
    return g, t.copy()


def _check(gb, tb, code, ctx, thresholds=synth.THRESHOLDS):
    got = P.signature(to_device(gb, code), to_device(tb, code), synth.BINS, thresholds)
    assert_parity(got, oracle_sig(gb, tb, code, synth.BINS, thresholds), ctx)
    return got


@pytest.mark.parametrize("code", [0, 1, 2])
@pytest.mark.parametrize("n", [1, 255, 1023, 1024, 2047, 2049, 4095, 4096, 5121, 8193, 70001, (1 << 20) + 3])
def test_rectified(code, n):
    for eps in (0.0, 2e-3):
        gb, tb = _relu(n, code, 100 * n + code, eps)
        _check(gb, tb, code, f"relu n={n} eps={eps}")
        _check(gb, tb, code, f"relu ladder n={n} eps={eps}", LADDER)


@pytest.mark.parametrize("code", [0, 1, 2])
def test_signed_zeros_and_equal_vectors(code):
    """Zeros of either sign against each other, all-zero goldens before the
    first nonzero one, bit-equal vectors with zeros, infinite and NaN goldens."""
    n = 40000
    sp = _SPECIALS[code]
    rng = np.random.default_rng(code)
    gb, tb = _relu(n, code, 7 + code)
    tb = gb.copy()
    gb[:12000] = tb[:12000] = sp["zero"]
    _check(gb, tb, code, "zeros first")
    for name in ("nzero", "sub", "inf", "nan", "big"):
        g, t = gb.copy(), tb.copy()
        idx = rng.integers(0, n, 20)
        t[idx] = sp[name]
        _check(g, t, code, f"test {name}")
        g[idx] = sp[name]
        _check(g, t, code, f"both {name}")
        t[idx] = sp["nzero"]
        _check(g, t, code, f"golden {name}, test -0")
    _check(np.full(n, sp["zero"], gb.dtype), np.full(n, sp["nzero"], gb.dtype), code, "+0 / -0")
    _check(np.full(n, sp["nzero"], gb.dtype), np.full(n, sp["nzero"], gb.dtype), code, "-0 / -0")


@pytest.mark.parametrize("code", [0, 1, 2])
@pytest.mark.parametrize("per_vec", [1, 31, 32, 33, 64, 65, 200])
def test_elements_per_vector(code, per_vec):
    """per_vec elements of every wave's vector need the generic path, in full
    chunks and in a ragged one: below, at and above the 64 worked at once."""
    n = 3 * (1 << 15) + 777
    gb, tb = special_pair(n, code, seed=per_vec + code, special_frac=0.0)
    rng = np.random.default_rng(per_vec)
    span = 64 * VEC[code]
    names = list(_SPECIALS[code].values())
    for k in range(0, n, span):
        idx = k + rng.choice(min(span, n - k), min(per_vec, n - k), replace=False)
        idx = idx[idx < n]
        half = len(idx) // 2
        tb[idx[:half]] = rng.choice(names, half)
        gb[idx[half:]] = rng.choice(names, len(idx) - half)
    _check(gb, tb, code, f"{per_vec} per vector")
    # the first element of a vector is not valid: argmax of an all-zero error
    gb, tb = special_pair(n, code, seed=1, special_frac=0.0)
    tb = gb.copy()
    tb[::span] = _SPECIALS[code]["nan"]
    _check(gb, tb, code, "NaN first, otherwise equal")


@pytest.mark.parametrize("code", [0, 1, 2])
@pytest.mark.parametrize("off", [(1, 0), (0, 1), (1, 1), (3, 5), (7, 2)])
def test_unaligned_offsets(code, off):
    """Slices that start anywhere give the record of the aligned tensors."""
    n = 150003
    gb, tb = special_pair(n + 8, code, seed=3 + code)
    og, ot = off
    g, t = gb[og:og + n], tb[ot:ot + n]
    dg, dt = to_device(gb, code)[og:og + n], to_device(tb, code)[ot:ot + n]
    got = P.signature(dg, dt, synth.BINS, synth.THRESHOLDS)
    assert records_equal(got, _check(g, t, code, f"offsets {off}"))
    top = P.topk_mean(dg, dt)
    assert top == P.topk_mean(to_device(g.copy(), code), to_device(t.copy(), code))


@pytest.mark.parametrize("kind", [(0, 3), (0, 1), (0, 2), (1, 0), (2, 0), (1, 3), (2, 3)])
def test_mixed_rectified(kind):
    """Zero goldens in mixed pairs, tiny binary64 tests against them included."""
    G, T = kind
    rng = np.random.default_rng(10 * G + T)
    for n in (1000, 4096, 33333):
        x = np.maximum(rng.standard_normal(n), 0.0)
        y = x * (1 + 1e-5 * rng.standard_normal(n))
        z = np.flatnonzero(x == 0)
        y[z[::50]] = rng.choice([1e-3, -1e-30, 5e-324, -0.0, np.nan, np.inf, 1e-310], len(z[::50]))
        gb = float_to_bits(x, G).copy()
        tb = y if T == 3 else float_to_bits(y, T).copy()
        td = torch.from_numpy(tb).cuda() if T == 3 else to_device(tb, T)
        got = P.signature_mixed(to_device(gb, G), td, synth.BINS, LADDER)
        ref = oracle.signature_mixed(gb, tb, gdtype=G, tdtype=T, bins=synth.BINS, thresholds=LADDER)
        assert_parity(got, ref, f"kind {kind} n={n}")
