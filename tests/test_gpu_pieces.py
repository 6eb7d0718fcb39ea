"""Chunks whose sums are formed piece by piece (2^16 elements and more): a call
of few chunks gives each piece a block, a larger one works them in turn.  The
records are the same bits either way, and those of the oracle, at the edges of
pieces and chunks, with and without special values."""
from __future__ import annotations


import pytest
import torch

import paper_2609_13544_amd as P
import synth
from tests.parity import assert_parity, chunk_count, oracle_sig, special_pair, to_device

pytestmark = pytest.mark.gpu

FEW = 1536                            # chunks of a call up to which pieces get blocks
M = 1 << 22


@pytest.mark.parametrize("n,code,frac", [
    (M - 1, 0, 0.0), (M, 0, 1e-4), (M, 1, 0.0), (M + 1, 2, 1e-4), (M + (3 << 14), 1, 1e-4), (M + (1 << 16) + 4097, 0, 1e-3),
    (2 * M + 12345, 2, 0.0), (4 * M, 1, 0.0), (4 * M + 1, 0, 1e-5),
])
def test_pieces(n, code, frac):
    gb, tb = special_pair(n, code, seed=n + code, special_frac=frac)
    g, t = to_device(gb, code), to_device(tb, code)
    lone = P.signature(g, t, synth.BINS, synth.THRESHOLDS)
    assert_parity(lone, oracle_sig(gb, tb, code, synth.BINS, synth.THRESHOLDS))
    many = FEW // chunk_count(n) + 1
    for rec in P.signature_batched([(g, t)] * many, synth.BINS, synth.THRESHOLDS):
        assert repr(rec) == repr(lone)
    small = (g[:5000], t[:5000])
    few = P.signature_batched([small, (g, t), small], synth.BINS, synth.THRESHOLDS)
    assert repr(few[1]) == repr(lone)
    for count in (1, many):
        d_out = torch.zeros(count * P.SIG_BYTES, dtype=torch.uint8, device="cuda")
        P.signature_batched_noalloc([(g, t)] * count, d_out, synth.BINS, synth.THRESHOLDS)
        torch.cuda.synchronize()
        for rec in P.decode_records(d_out, count, nthr=len(synth.THRESHOLDS)):
            assert repr(rec) == repr(lone)
