"""The edit distance's first pass over fewer diagonals: pairs that cannot end within them
leave it early, whatever their letters, and every distance equals the oracle's -- of pairs
that leave rightly, that leave although they would have ended there, that stay and outgrow
it, and of unequal lengths."""
import numpy as np
import pytest

from paper_2607_06225_amd import workloads as W
from tests.parity import compare, oracle_batch

pytestmark = pytest.mark.gpu


def pair(rng, kind, L, symbols):
    r = rng.integers(0, symbols, size=L).astype(np.uint8)
    other = ((r + 1 + rng.integers(0, symbols - 1, size=L)) % symbols).astype(np.uint8)
    at = np.arange(L)
    if kind == 0:  # unrelated
        return rng.integers(0, symbols, size=L).astype(np.uint8), r
    if kind == 1:  # a first seventh unlike, then the same
        return np.where(at < L // 7, other, r), r
    if kind == 2:  # the same, then a tail with no letter of the other
        return np.where(at < L // 5, r, 0).astype(np.uint8), np.where(at < L // 5, r, 1).astype(np.uint8)
    if kind == 3:  # close
        return np.where(rng.random(L) < 0.05, other, r), r
    if kind == 4:  # another length, the same letters
        return r[: L - L // 9], r
    return other, r  # no letter equal in place


@pytest.mark.parametrize("symbols", [2, 4, 5, 20])
@pytest.mark.parametrize("n,L", [(5200, 1500), (1100, 4000)])
def test_pairs_leave_the_first_pass_early(symbols, n, L):
    import torch
    from paper_2607_06225_amd import aln
    assert torch.cuda.is_available()
    rng = np.random.default_rng(symbols + L)
    m = np.full((symbols, symbols), -1, dtype=np.int32)
    np.fill_diagonal(m, 0)
    ctx = aln.Context(0)
    ctx.set_profiling(True)
    for kinds in (range(6), (0,)):
        some = [pair(rng, k, L - 37 * c, symbols) for c in range(3) for k in kinds]
        one = W.pack_pairs([p[0] for p in some], [p[1] for p in some], m, 0, -1, W.GLOBAL, W.SEARCH,
                           name=f"cap_{symbols}_{L}")
        idx = np.arange(n) % one.n
        b = W.Batch(one.name, one.q, one.q_off[idx], one.q_len[idx], one.r, one.r_off[idx],
                    one.r_len[idx], m, 0, -1, W.GLOBAL, W.SEARCH, 0, 0, False)
        print(f"[gpu] {b.name} {list(kinds)}", flush=True)
        ctx.kernel_times()
        res, _ = aln.align(ctx, b)
        ms = {k: v[0] for k, v in ctx.kernel_times().items()}
        assert "search_wide" in ms  # there is such a pass
        assert compare(one, res[:one.n], None, oracle_batch(one)) == []
        assert np.array_equal(res["score"], res["score"][:one.n][idx])
        assert np.array_equal(res["cells"], res["cells"][:one.n][idx])
        if symbols == 20 and len(kinds) == 1:  # all of them searched twice: 0.4 of the time before
            assert ms["search"] < 0.2 * ms["search_wide"]
    ctx.set_profiling(False)
    ctx.close()
