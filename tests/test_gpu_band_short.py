"""Narrow bands over short pairs beside ones of 128 rows and more: all of them on the band
strips, in one launch, from one row on (in large batches from 32), equal to the oracle."""
import numpy as np
import pytest
import torch

from paper_2607_06225_amd import aln, workloads as W
from tests.parity import compare, oracle_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available()
    c = aln.Context(0)
    c.set_tuning({"valid": 0})
    yield c
    c.close()


@pytest.mark.parametrize("mode", [W.GLOBAL, W.LOCAL, W.EXTEND])
@pytest.mark.parametrize("letters,n", [(20, 40), (20, 1500), (4, 15)])
@pytest.mark.parametrize("w", [0, 3, 17, 64, 127])
def test_short_pairs_beside_longer_ones(ctx, letters, n, w, mode):
    rng = np.random.default_rng(n + w)
    qs, rs = [], []
    for k in range(n):
        M = (128, 200, 1, 2, 31, 32, 33, 63, 64, 65, 127, 90)[k] if k < 12 else int(rng.integers(1, 180))
        N = max(1, int(M * (1.0, 1.15, 0.85, 2.5, 0.3)[k % 5]) + k % 3)
        r = rng.integers(0, letters, size=N).astype(np.uint8)
        q = rng.integers(0, letters, size=M).astype(np.uint8)
        at = (np.arange(M) * N) // M
        near = rng.random(M) < 0.9
        q[near] = r[at[near]]
        qs.append(q)
        rs.append(r)
    m, go, ge = (W.dna_matrix(1, -2), -2, -1) if letters == 4 else (W.protein_matrix(202), -11, -1)
    for cigar in (False, True):
        b = W.pack_pairs(qs, rs, m, go, ge, mode, W.BAND, band_w=w, want_cigar=cigar,
                         name=f"short_w{w}_{letters}")
        sid = ctx.set_scoring(m, go, ge)
        p = ctx.plan(sid, b.q_len, b.r_len, mode, W.BAND, w, 0, want_cigar=cigar)
        L, T = p.describe()
        p.close()
        # antidiagonals only for pairs under 32 rows of large batches (and full matrices
        # elsewhere: pairs no longer than the band)
        small = [t for t in T if L[t["launch"]]["family"] == "diag_band"]
        assert all(n > 1024 and b.q_len[t["pair"]] < 32 for t in small)
        assert any(l["family"] == "band_strip" for l in L)
        print(f"[gpu] {b.name} n={n} mode={mode} cigar={cigar}", flush=True)
        res, cig = aln.align(ctx, b)
        assert compare(b, res, cig, oracle_batch(b)) == []
