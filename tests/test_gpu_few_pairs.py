"""Small batches of full matrices, where a pair's strips share a workgroup of four or
eight wavefronts: lengths on both sides of each choice, equal to the oracle; and the
choice that keeps within the workspace of a call without allocation."""
import numpy as np
import pytest

from paper_2607_06225_amd import workloads as W
from tests.parity import compare, oracle_batch


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2607_06225_amd import aln
    assert torch.cuda.is_available()
    c = aln.Context(0)
    yield c
    c.close()


@pytest.mark.gpu
@pytest.mark.parametrize("longest", [511, 512, 513, 640, 641, 1024, 1025, 1408, 1409, 2038])
@pytest.mark.parametrize("mode,letters", [(W.GLOBAL, 4), (W.LOCAL, 20), (W.EXTEND, 4)])
def test_few_full_matrices(ctx, longest, mode, letters):
    from paper_2607_06225_amd import aln
    rng = np.random.default_rng(longest + mode)
    qs, rs = [], []
    for M, N in ((longest, longest), (longest, 70), (90, min(longest, 2000)), (longest // 2, longest),
                 (longest - 1, longest // 3)):
        q = rng.integers(0, letters, size=M).astype(np.uint8)
        r = rng.integers(0, letters, size=N).astype(np.uint8)
        k = min(M, N) - 5
        r[:k] = q[:k]
        r[rng.random(N) < 0.1] = 1
        qs.append(q)
        rs.append(r)
    m = W.dna_matrix(2, -4) if letters == 4 else W.protein_matrix(202)
    b = W.pack_pairs(qs, rs, m, -4, -2, mode, W.FULL, want_cigar=True,
                     name=f"few{longest}_{mode}")
    print(f"[gpu] {b.name}", flush=True)
    res, cig = aln.align(ctx, b)
    assert compare(b, res, cig, oracle_batch(b)) == []


def test_codes_stay_within_the_fixed_workspace():
    """200 pairs of 512 x 1 250: 63 MiB of codes at eight rows a lane, more at two."""
    from paper_2607_06225_amd import aln
    c = aln.Context.host()
    sid = c.set_scoring(W.dna_matrix(2, -4), -4, -2)
    p = c.plan(sid, np.full(200, 512, np.int32), np.full(200, 1250, np.int32), W.GLOBAL, W.FULL, 0, 0,
               want_cigar=True)
    assert 60 << 20 < p.workspace_bytes <= aln.NOALLOC_WORKSPACE_BYTES
    p.close()
    c.close()
