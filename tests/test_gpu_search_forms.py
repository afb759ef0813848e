"""The score-major search with 1, 2, 4 and 8 wavefronts a pair (chosen by how many
pairs a CU holds), codes packed two bits each (four symbols) or in bytes (more), and
penalties with and without a common divisor: whole numbers, equal to the oracle."""
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


@pytest.mark.parametrize("symbols", [4, 5])
@pytest.mark.parametrize("pen", [None, (4, 6, 2), (6, 6, 3), (5, 0, 5), (2, 3, 1)])
@pytest.mark.parametrize("n,longest", [(4200, 40), (2200, 70), (800, 130), (40, 700)])
def test_search_forms(ctx, symbols, pen, n, longest):
    from paper_2607_06225_amd import aln
    rng = np.random.default_rng(n + symbols)
    qs, rs = [], []
    for k in range(n):
        r = rng.integers(0, symbols, size=int(rng.integers(0, longest + 1))).astype(np.uint8)
        q = r.copy()
        for _ in range(int(rng.integers(0, 5)) if k % 7 else 0):
            at = int(rng.integers(0, len(q) + 1))
            kind = int(rng.integers(0, 3))
            if kind == 0:
                q = np.insert(q, at, rng.integers(0, symbols)).astype(np.uint8)
            elif at < len(q):
                q = np.delete(q, at) if kind == 1 else q.copy()
                if kind == 2:
                    q[at] = (q[at] + 1) % symbols
        if k % 11 == 0:  # unrelated, of another length
            q = rng.integers(0, symbols, size=int(rng.integers(0, longest + 1))).astype(np.uint8)
        qs.append(q)
        rs.append(r)
    x, o, e = pen or (1, 0, 1)
    m = np.full((symbols, symbols), -x, dtype=np.int32)
    np.fill_diagonal(m, 0)
    b = W.pack_pairs(qs, rs, m, -o, -e, W.GLOBAL, W.SEARCH, name=f"forms_{symbols}_{pen}_{n}")
    print(f"[gpu] {b.name}", flush=True)
    res, _ = aln.align(ctx, b)
    assert compare(b, res, None, oracle_batch(b)) == []


def test_edit_distance_outgrows_capped_rows(ctx):
    """Long pairs of a large batch first run with rows of some 0.55 of the longest length's
    diagonals a side: pairs with no letter in common, whose distance is their length, and
    ones close to the cap are right, and nothing is left marked in the flags."""
    from paper_2607_06225_amd import aln
    rng = np.random.default_rng(77)
    qs, rs = [], []
    for k in range(2700):
        L = 1500 - k // 4 if k < 12 else int(rng.integers(0, 60))
        q = rng.integers(0, 2, size=L).astype(np.uint8)
        if k % 4 == 0:
            r = q + 2  # no letter in common: distance L
        elif k % 4 == 1:
            r = q.copy()
            r[: int(0.55 * L) + 8] += 2  # at the cap
        elif k % 4 == 2:
            r = rng.integers(0, 2, size=max(0, L - 40)).astype(np.uint8)
        else:
            r = q.copy()
        qs.append(q)
        rs.append(r.astype(np.uint8))
    b = W.pack_pairs(qs, rs, W.dna_matrix(0, -1), 0, -1, W.GLOBAL, W.SEARCH, name="outgrown")
    print(f"[gpu] {b.name}", flush=True)
    res, _ = aln.align(ctx, b)
    assert compare(b, res, None, oracle_batch(b)) == []
    assert int(res["score"][0]) == -1500 and not res["flags"].any()
    one, _ = aln.align(ctx, b, graph=True)
    assert np.array_equal(res, one)
