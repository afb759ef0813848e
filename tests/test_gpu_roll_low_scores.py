"""Short queries against references so long, or gaps so steep, that cells of the full
matrix score below -32 768, as rolling row blocks: EXTEND's best cell (and GLOBAL's
score) equal to the oracle's, with and without paths."""
import numpy as np
import pytest

from paper_2607_06225_amd import workloads as W
from tests.parity import compare, oracle_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2607_06225_amd import aln
    assert torch.cuda.is_available()
    c = aln.Context(0)
    c.set_tuning({"valid": 0})
    yield c
    c.close()


@pytest.mark.parametrize("mode", [W.EXTEND, W.GLOBAL])
@pytest.mark.parametrize("n,M,N,go,ge", [(24, 150, 20000, -4, -2), (24, 100, 65535, 0, -1),
                                         (300, 160, 400, -4, -200), (300, 120, 330, -1024, -1024),
                                         (300, 33, 64, 0, -1000)])
def test_low_scores(ctx, n, M, N, go, ge, mode):
    from paper_2607_06225_amd import aln
    rng = np.random.default_rng(M + N)
    qs, rs = [], []
    for k in range(n):
        m, l = M - k % 7, N - 3 * (k % 5)
        q = rng.integers(0, 4, size=m).astype(np.uint8)
        r = rng.integers(0, 4, size=l).astype(np.uint8)
        if k % 3:  # a planted start (k % 3 == 1: of the whole query)
            keep = min(m if k % 3 == 1 else m // 2, l)
            r[:keep] = q[:keep]
        qs.append(q)
        rs.append(r)
    for cigar in (False, True):
        b = W.pack_pairs(qs, rs, W.dna_matrix(2, -4), go, ge, mode, W.FULL, want_cigar=cigar,
                         name=f"low{M}x{N}_{ge}")
        sid = ctx.set_scoring(b.matrix, b.gap_open, b.gap_extend)
        p = ctx.plan(sid, b.q_len, b.r_len, mode, W.FULL, 0, 0, want_cigar=cigar)
        L, _ = p.describe()
        p.close()
        assert {l["family"] for l in L} == {"roll_i32"}
        print(f"[gpu] {b.name} n={n} cigar={cigar}", flush=True)
        res, cig = aln.align(ctx, b)
        assert compare(b, res, cig, oracle_batch(b)) == []
