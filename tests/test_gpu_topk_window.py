"""GPU parity of the top-k mean where its steps change: pairs at and around the
size that one block settles, windows that hold T, miss it, span a binade's end
or have no nonzero error, keys that repeat or do not, buffers that are too
small (digit passes), against the oracle; tolerances as in test_gpu_topk.py."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2609_13544_amd as P
from tests.parity import float_to_bits, special_pair, to_device
from tests.test_gpu_topk import assert_topk, same_record

pytestmark = pytest.mark.gpu

SMALL = 1 << 14                       # errors that one block settles


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    P.lib()
    assert oracle.lib()
    yield
    P.topk_set_entry_capacity(-1, -1)
    torch.cuda.synchronize()


def _data(name, n, code, rng):
    g = rng.standard_normal(n)
    if name == "repeating":           # errors of a few last places
        return g, g * (1 + {0: 1e-7, 1: 1e-3, 2: 1e-2}[code] * rng.standard_normal(n))
    if name == "distinct":            # hardly any error twice (f32)
        return g, g + 1e-2 * rng.standard_normal(n)
    if name == "binade end":          # T sits at a power of two
        return np.zeros(n), np.where(rng.random(n) < 0.1, 2.0, 1.999) * (1 + 1e-3 * (rng.random(n) < 0.2))
    if name == "mostly zero":         # the k-th error among the zeros, by a hair or by far
        return g, np.where(rng.random(n) < 0.0995, g * 1.5, g)
    if name == "zero":
        return g, np.where(rng.random(n) < 0.02, g + 1.0, g)
    if name == "rows":                # whole stretches alike: the sample misjudges its rank
        row = np.repeat(10.0 ** rng.uniform(-6, 3, n // 3000 + 1), 3000)[:n]
        return g, g + row * rng.standard_normal(n)
    if name == "tail":                # the largest errors in one place
        return g, np.where(np.arange(n) >= n - n // 9, g * 3.0, g * (1 + 1e-5 * rng.standard_normal(n)))
    raise ValueError(name)


@pytest.mark.parametrize("code", [0, 1, 2])
@pytest.mark.parametrize("n", [1, 7, SMALL - 1, SMALL, SMALL + 1, 2 * SMALL + 3, 300007])
@pytest.mark.parametrize("name", ["repeating", "distinct", "binade end", "mostly zero", "zero", "rows", "tail"])
def test_windows(name, n, code):
    rng = np.random.default_rng(n + code)
    G, T = _data(name, n, code, rng)
    gb, tb = float_to_bits(G, code).copy(), float_to_bits(T, code).copy()
    g, t = to_device(gb, code), to_device(tb, code)
    for num, den in ((1, 10), (1, 1000), (1, 1)):
        P.topk_set_entry_capacity(-1, -1)
        got = P.topk_mean(g, t, num, den)
        assert_topk(got, oracle.topk(gb, tb, dtype=code, num=num, den=den), f"{name} n={n} {num}/{den}")
        P.topk_set_entry_capacity(0, 0)
        assert same_record(P.topk_mean(g, t, num, den), got), f"{name} n={n} {num}/{den}: digit passes differ"


@pytest.mark.parametrize("caps", [(0, 300), (5, -1), (-1, 0), (-1, 256)])
def test_partly_filled_buffers(caps):
    """Some pairs of a batch fit, others do not; every record is the lone call's."""
    rng = np.random.default_rng(3)
    pairs = []
    for k, n in enumerate((SMALL + 1, 70001, 1 << 18, 5, 200003)):
        gb, tb = special_pair(n, k % 3, seed=k, special_frac=1e-3)
        if k == 2:
            tb = float_to_bits(rng.standard_normal(n), 2).copy()
        pairs.append((to_device(gb, k % 3), to_device(tb, k % 3)))
    P.topk_set_entry_capacity(-1, -1)
    ref = [P.topk_mean(*p) for p in pairs]
    P.topk_set_entry_capacity(*caps)
    for a, b in zip(P.topk_mean_batched(pairs), ref):
        assert same_record(a, b)
