"""A pair with a code past the alphabet is a bad symbol, whatever else a kernel finds: end
cells that a band does not reach, regions wider than every window."""
import numpy as np
import pytest
import torch

from paper_2607_06225_amd import aln, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("letters,n,L,families", [
    (20, 3, 60, {"diag_band"}), (20, 40, 200, {"band_strip"}), (4, 40, 200, {"band_roll"})])
def test_unreachable_band(letters, n, L, families):
    assert torch.cuda.is_available()
    rng = np.random.default_rng(L)
    qs = [rng.integers(0, letters, size=L).astype(np.uint8) for _ in range(n)]
    rs = [rng.integers(0, letters, size=2 * L + k % 3).astype(np.uint8) for k in range(n)]
    for k in (0, n - 1):
        qs[k][5] = letters
    m = np.where(np.eye(letters, dtype=bool), 1, -2).astype(np.int32)
    b = W.pack_pairs(qs, rs, m, -2, -1, W.GLOBAL, W.BAND, band_w=0, name=f"bad{letters}_{n}")
    check(b, families, 1)  # unreachable: two columns a row


def test_too_wide_region():
    rng = np.random.default_rng(1)
    qs, rs = ([rng.integers(0, 4, size=2600).astype(np.uint8) for _ in range(6)] for _ in range(2))
    for k in (0, 5):
        rs[k][2599] = 4
    for prune, X in ((W.XDROP, 30000), (W.ZDROP, 30000)):
        check(W.pack_pairs(qs, rs, W.dna_matrix(2, -4), -4, -2, W.EXTEND, prune, xdrop=X,
                           name=f"bad_wide{prune}"), None, 4)


def check(b, families, status):
    ctx = aln.Context(0)
    sid = ctx.set_scoring(b.matrix, b.gap_open, b.gap_extend)
    p = ctx.plan(sid, b.q_len, b.r_len, b.mode, b.prune, b.band_w, b.xdrop)
    if families:
        assert {l["family"] for l in p.describe()[0]} == families
    p.close()
    print(f"[gpu] {b.name}", flush=True)
    res, _ = aln.align(ctx, b)
    ctx.close()
    want = np.full(b.n, status)
    want[[0, -1]] = 3
    assert res["status"].tolist() == want.tolist()
