"""The lanes kernel's forms by batch size: sixteen lanes a side for small
batches (the other X-drop tests), eight and four for larger ones, and Z-drop's
eight lanes over 128 cells, bit-exact against the oracle.  A batch is some
distinct pairs repeated until it is large enough for the form."""
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


def distinct(rng, n):
    """Similar and unrelated pairs, empty ones, ones much longer on one side,
    and pairs with a long insertion (regions that drift and outgrow a window)."""
    st = W.Stream(int(rng.integers(1, 1 << 30)), 9)
    qs, rs = [], []
    for p in range(n):
        N = int(rng.integers(0, 260)) if p % 40 else int(rng.integers(600, 1300))
        ref = rng.integers(0, 4, size=N).astype(np.uint8)
        kind = p % 5
        if kind == 0:
            q = rng.integers(0, 4, size=int(rng.integers(0, 260))).astype(np.uint8)
        elif kind == 1 and N > 40:
            at, gap = int(rng.integers(10, N - 10)), int(rng.integers(5, 70))
            q = np.concatenate([ref[:at], rng.integers(0, 4, size=gap).astype(np.uint8), ref[at:]])
        elif kind == 2 and N > 60:
            at = int(rng.integers(10, N // 2))
            q = np.concatenate([ref[:at], ref[at + int(rng.integers(5, N // 2)):]])
        else:
            q = W.mutate(ref, float(rng.uniform(0.01, 0.3)), 2, 1, 1, 4, st)
        qs.append(q)
        rs.append(ref)
    return qs, rs


def sides_of(plan):
    L, _ = plan.describe()
    return [(l["family"], l["sides"]) for l in L]


@pytest.mark.parametrize("prune,X,cigar,n,form", [
    (W.XDROP, 100, False, 16384, ("xdrop_lanes", 4)),
    (W.XDROP, 100, False, 16385, ("xdrop_lanes", 8)),
    (W.XDROP, 131, False, 65536, ("xdrop_lanes", 8)),
    (W.XDROP, 60, False, 65537, ("xdrop_lanes", 16)),
    (W.XDROP, 131, True, 20000, ("xdrop_lanes_tb", 8)),
    (W.XDROP, 100, True, 66000, ("xdrop_lanes_tb", 16)),
    (W.ZDROP, 40, False, 16384, ("zdrop", 1)),
    (W.ZDROP, 100, False, 16385, ("zdrop_lanes", 8)),
    (W.ZDROP, 180, False, 20000, ("zdrop_lanes", 8)),
])
def test_form_by_batch_size(ctx, prune, X, cigar, n, form):
    import torch
    from paper_2607_06225_amd import aln
    print(f"[gpu] {form} n={n} X={X}", flush=True)
    K = 1000
    qs, rs = distinct(np.random.default_rng(n + X), K)
    one = W.pack_pairs(qs, rs, W.dna_matrix(2, -4), -4, -2, W.EXTEND, prune, xdrop=X,
                       want_cigar=cigar)
    idx = np.arange(n) % K
    b = W.Batch(one.name, one.q, one.q_off[idx], one.q_len[idx], one.r, one.r_off[idx],
                one.r_len[idx], one.matrix, -4, -2, W.EXTEND, prune, 0, X, cigar)
    sid = ctx.set_scoring(b.matrix, -4, -2)
    plan = ctx.plan(sid, b.q_len, b.r_len, b.mode, b.prune, 0, X, want_cigar=cigar)
    assert sides_of(plan) == [form]
    db, buf = aln.DeviceBatch(b), aln.Buffers(plan)
    ctx.execute(plan, db, buf.ws, buf.res, buf.cigar)
    torch.cuda.synchronize()
    res = buf.results(n)
    cig = buf.cigars(res) if cigar else None
    ores = oracle_batch(one)
    for lo in (0, n - K):  # the longest's and the last's round
        rows = np.arange(lo, lo + K)
        assert compare(one, res[rows], [cig[r] for r in rows] if cigar else None, ores,
                       idx=idx[rows]) == []
    for f in ("score", "q_end", "r_end", "cells", "status", "flags", "cigar_len", "q_begin",
              "r_begin"):
        assert np.array_equal(res[f], res[f][:K][idx]), f
    if prune == W.ZDROP:  # the flag marks what outgrew 250 diagonals in either form
        small = b.subset(np.arange(K))
        r1, _ = aln.align(ctx, small, scoring_id=sid)
        assert np.array_equal(r1["flags"], res["flags"][:K])
        if X == 180:
            assert (r1["flags"] != 0).any()
    plan.close()
