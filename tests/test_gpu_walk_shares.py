"""Walks by several wavefronts a pair (shares of the rows joined where their
paths agree) against the oracle's CIGARs: paths far off the guessed line, long
gaps over a share's rows, runs longer than the shares, and paths of more words
than a share's buffer holds."""
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


def far(rng, n, kind):
    """A pair of about n bases whose path leaves the straight line."""
    ref = rng.integers(0, 4, size=n).astype(np.uint8)
    junk = lambda k: rng.integers(0, 4, size=k).astype(np.uint8)  # noqa: E731
    st = W.Stream(int(rng.integers(1, 1 << 30)), 5)
    if kind == "same":  # one run of matches
        return ref, ref.copy()
    if kind == "unrelated":
        return junk(n + 7), ref
    if kind == "dense":  # words a share's buffer cannot hold
        return W.mutate(ref, 0.45, 2, 1, 1, 4, st), ref
    if kind == "insert":  # down a column over whole shares, then back by a deletion
        return np.concatenate([ref[: n // 3], junk(n // 4), ref[n // 3: -n // 4]]), ref
    if kind == "delete":
        return np.concatenate([ref[: n // 5], ref[n // 2:], junk(n // 4)]), ref
    return W.mutate(ref, 0.12, 3, 5, 4, 4, st), ref  # "edits"


KINDS = ["same", "unrelated", "dense", "insert", "delete", "edits"]


@pytest.mark.parametrize("mode", [W.GLOBAL, W.EXTEND])
@pytest.mark.parametrize("w,lo,hi,n", [(256, 2100, 6000, 18), (200, 600, 3000, 600),
                                       (64, 300, 2500, 1100), (70, 2100, 9000, 18),
                                       (1500, 900, 1400, 18), (1500, 500, 620, 18)])
def test_shares(ctx, mode, w, lo, hi, n):
    """w = 64, 70: rolling blocks; 200, 256: band strips; 1 500: full-matrix
    pairs on band strips.  n and hi choose 4, 8 or 16 wavefronts."""
    from paper_2607_06225_amd import aln
    rng = np.random.default_rng(w + n + mode)
    base = [far(rng, int(rng.integers(lo, hi)), KINDS[k % len(KINDS)]) for k in range(min(n, 60))]
    base = [(q[: max(1, int(len(r) * 1.25))], r) for q, r in base]
    one = W.pack_pairs([q for q, _ in base], [r for _, r in base], W.dna_matrix(2, -4), -4, -2,
                       mode, W.FULL if w == 1500 else W.BAND, band_w=0 if w == 1500 else w,
                       want_cigar=True, name=f"shares_w{w}")
    K = one.n
    idx = np.arange(n) % K
    b = W.Batch(one.name, one.q, one.q_off[idx], one.q_len[idx], one.r, one.r_off[idx],
                one.r_len[idx], one.matrix, -4, -2, mode, one.prune, one.band_w, 0, True)
    print(f"[gpu] {b.name} n={n} mode={mode}", flush=True)
    res, cig = aln.align(ctx, b)
    ores = oracle_batch(one)
    for lo_ in (0, n - K):
        rows = np.arange(lo_, lo_ + K)
        assert compare(one, res[rows], [cig[r] for r in rows], ores, idx=idx[rows]) == []
    assert np.array_equal(res["cigar_len"], res["cigar_len"][:K][idx])
