"""Rolling row blocks on bands whose best paths run along an edge of the band, from the
shape where a lane's next block starts as soon as it has left the one before to shapes a
few columns longer: equal to the oracle, with and without paths."""
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


def along(rng, M, N, w, edge, slack):
    """A pair whose rows match the column `slack` inside the band's edge (-1 left, 1 right)."""
    q = rng.integers(0, 4, size=M).astype(np.uint8)
    r = rng.integers(0, 4, size=N).astype(np.uint8)
    for i in range(1, M + 1):
        j = i * N // M + edge * (w - slack)
        if 1 <= j <= N:
            q[i - 1] = r[j - 1]
    return q, r


@pytest.mark.parametrize("mode", [W.GLOBAL, W.LOCAL, W.EXTEND])
@pytest.mark.parametrize("w,M,lens", [(15, 600, range(576, 606)), (12, 600, range(476, 490)),
                                      (14, 1000, range(904, 916)), (87, 1000, range(984, 1006)),
                                      (60, 1500, range(845, 875))])
def test_paths_along_the_band(ctx, w, M, lens, mode):
    from paper_2607_06225_amd import aln
    rng = np.random.default_rng(1000 * w + mode)
    qs, rs = [], []
    for N in lens:
        for edge in (-1, 1):
            for slack in (0, 1):
                q, r = along(rng, M, N, w, edge, slack)
                qs.append(q)
                rs.append(r)
    for cigar in (False, True):
        b = W.pack_pairs(qs, rs, W.dna_matrix(1, -2), -2, -1, mode, W.BAND, band_w=w,
                         want_cigar=cigar, name=f"edge_w{w}_m{mode}")
        sid = ctx.set_scoring(b.matrix, b.gap_open, b.gap_extend)
        p = ctx.plan(sid, b.q_len, b.r_len, mode, W.BAND, w, 0, want_cigar=cigar)
        L, _ = p.describe()
        p.close()
        assert "band_roll" in {l["family"] for l in L}
        print(f"[gpu] {b.name} n={b.n} cigar={cigar}", flush=True)
        res, cig = aln.align(ctx, b)
        assert compare(b, res, cig, oracle_batch(b)) == []
