"""Z-drop sides by how far from the best diagonal Z lets a region reach: which form runs
first and which wider passes follow, results equal to the oracle's."""
import numpy as np
import pytest
import torch

from paper_2607_06225_amd import aln, workloads as W
from tests.parity import compare, oracle_batch


@pytest.mark.parametrize("ge,Z,family", [(-2, 100, "zdrop_lanes"), (-2, 184, "zdrop_lanes"),
                                         (-2, 185, "zdrop"), (-2, 700, "zdrop"), (-1, 40, "zdrop"),
                                         (-3, 364, "zdrop_lanes"), (-3, 365, "zdrop")])
def test_first_form_of_large_batches(ge, Z, family):
    c = aln.Context.host()
    sid = c.set_scoring(W.dna_matrix(2, -4), -4, ge)
    lens = np.full(20000, 400, np.int32)
    p = c.plan(sid, lens, lens, W.EXTEND, W.ZDROP, 0, Z)
    L, _ = p.describe()
    assert [l["family"] for l in L] == [family]
    p.close()
    c.close()


@pytest.mark.gpu
@pytest.mark.parametrize("cigar", [False, True])
@pytest.mark.parametrize("ge,Z,passes", [(-2, 60, 3), (-2, 184, 3), (-2, 185, 2), (-2, 254, 2),
                                         (-2, 700, 2), (-1, 30, 2), (-3, 364, 3), (-3, 365, 2)])
def test_wider_passes(ge, Z, passes, cigar):
    assert torch.cuda.is_available()
    rng = np.random.default_rng(Z - ge)
    qs, rs = [], []
    for k in range(24):
        r = rng.integers(0, 4, size=int(rng.integers(400, 1300))).astype(np.uint8)
        q = np.where(rng.random(r.size) < 0.03 * (k % 6), rng.integers(0, 4, size=r.size), r).astype(np.uint8)
        cut = int(rng.integers(0, 200)) if k % 2 else 0  # a long gap
        at = q.size // 2
        q = np.concatenate([q[:at], q[at + cut:], rng.integers(0, 4, size=60).astype(np.uint8)])
        qs.append(q)
        rs.append(np.concatenate([r, rng.integers(0, 4, size=40).astype(np.uint8)]))
    b = W.pack_pairs(qs, rs, W.dna_matrix(2, -4), -4, ge, W.EXTEND, W.ZDROP, xdrop=Z,
                     want_cigar=cigar, name=f"reach{Z}_{ge}")
    ctx = aln.Context(0)
    ctx.set_profiling(True)
    print(f"[gpu] {b.name}", flush=True)
    res, cig = aln.align(ctx, b)
    launches = ctx.kernel_times()["zdrop_wide"][1]
    ctx.set_profiling(False)
    ctx.close()
    assert launches == passes
    assert compare(b, res, cig, oracle_batch(b)) == []
