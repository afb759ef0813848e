"""Bands as wide as their type holds: the full matrix, equal to the oracle."""
import numpy as np
import pytest
import torch

from paper_2607_06225_amd import aln, workloads as W
from tests.parity import compare, oracle_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [W.GLOBAL, W.LOCAL, W.EXTEND])
@pytest.mark.parametrize("n", [1, 6, 400])
@pytest.mark.parametrize("w", [(1 << 31) - 1, (1 << 31) - 700, (1 << 28) + 1])
def test_widest_bands(n, w, mode):
    assert torch.cuda.is_available()
    rng = np.random.default_rng(n)
    qs, rs = [], []
    for k in range(n):
        r = rng.integers(0, 4, size=int(rng.integers(1, 900 if n < 100 else 200))).astype(np.uint8)
        q = np.where(rng.random(r.size) < 0.1, 2, r).astype(np.uint8)
        qs.append(np.concatenate([q, q[: k % 9]]))
        rs.append(r)
    b = W.pack_pairs(qs, rs, W.dna_matrix(2, -4), -4, -2, mode, W.BAND, band_w=w, want_cigar=True,
                     name=f"widest{w}_{n}")
    full = W.pack_pairs(qs, rs, W.dna_matrix(2, -4), -4, -2, mode, W.FULL, want_cigar=True)
    ctx = aln.Context(0)
    print(f"[gpu] {b.name} mode={mode}", flush=True)
    res, cig = aln.align(ctx, b)
    ctx.close()
    assert compare(full, res, cig, oracle_batch(full)) == []
