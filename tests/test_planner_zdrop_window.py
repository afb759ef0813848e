"""Z-drop tuned to the lanes form: 64-cell windows (sixteen sides a wavefront) where a
region's estimate fits one, else 128 cells (eight sides)."""
import numpy as np
import pytest

from paper_2607_06225_amd import aln, workloads as W


@pytest.mark.parametrize("extend,Z,sides", [(-2, 64, 16), (-2, 65, 8), (-3, 124, 16), (-3, 125, 8),
                                            (-1, 10, 8)])
def test_window_by_estimate(extend, Z, sides):
    c = aln.Context.host()
    c.set_tuning(dict(valid=True, sw16_rows=16, xdrop_rows=4, xdrop_sides=16))
    sid = c.set_scoring(W.dna_matrix(2, -4), -4, extend)
    lens = np.full(500, 300, np.int32)
    p = c.plan(sid, lens, lens, W.EXTEND, W.ZDROP, 0, Z)
    L, _ = p.describe()
    assert [(l["family"], l["sides"]) for l in L] == [("zdrop_lanes", sides)]
    p.close()
    c.close()
