"""X-drop and Z-drop sides whose lengths reach, just pass, or far pass what each window
holds, pruned so late that the whole matrix survives: only the passes that can be needed
are launched, and the results are the oracle's."""
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
    yield c
    c.close()


@pytest.mark.parametrize("span", [126, 127, 128, 250, 251, 252, 506, 507, 508, 1018, 1019, 1400])
@pytest.mark.parametrize("prune,X,cigar", [(W.XDROP, 100, False), (W.XDROP, 100, True),
                                           (W.XDROP, 5000, False), (W.XDROP, 5000, True),
                                           (W.ZDROP, 5000, False), (W.ZDROP, 5000, True)])
def test_every_width(ctx, span, prune, X, cigar):
    from paper_2607_06225_amd import aln
    rng = np.random.default_rng(span + X)
    qs, rs = [], []
    for M in (span // 2, span - 20, 20, span // 3):
        q = rng.integers(0, 4, size=M).astype(np.uint8)
        r = rng.integers(0, 4, size=span - M).astype(np.uint8)
        k = min(M, span - M)
        r[:k] = np.where(rng.random(k) < 0.2, r[:k], q[:k])
        qs.append(q)
        rs.append(r)
    # one batch a pair: the longest query and reference are that pair's
    for q, r in zip(qs, rs):
        b = W.pack_pairs([q], [r], W.dna_matrix(2, -4), -4, -2, W.EXTEND, prune, xdrop=X,
                         want_cigar=cigar, name=f"width{span}_{X}")
        res, cig = aln.align(ctx, b)
        assert compare(b, res, cig, oracle_batch(b)) == []
