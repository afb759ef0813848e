"""Which full matrices of large batches run as rolling row blocks: not rows a lane that few
pairs take beside longer ones, nor LOCAL pairs with paths and long references before
three pairs a SIMD (host planner; an MI355X has 1 024)."""
import numpy as np
import pytest

from paper_2607_06225_amd import aln, workloads as W


def tiles(ql, rl, mode, cigar):
    c = aln.Context.host()
    sid = c.set_scoring(W.dna_matrix(2, -4), -4, -2)
    p = c.plan(sid, np.asarray(ql, np.int32), np.asarray(rl, np.int32), mode, W.FULL, 0, 0,
               want_cigar=cigar)
    L, _ = p.describe()
    p.close()
    c.close()
    return {(l["family"], l["tile"]) for l in L}


@pytest.mark.parametrize("between,rolls", [(400, False), (511, False), (512, True)])
def test_few_pairs_of_a_height_stay_on_the_strips(between, rolls):
    ql = np.r_[np.full(4000, 60), np.full(between, 200), np.full(5000, 500)]
    got = tiles(ql, ql, W.LOCAL, True)
    assert ("roll_i32", 8) in got
    assert (("roll_i32", 16) in got) == rolls


def test_without_longer_pairs_every_height_rolls():
    ql = np.r_[np.full(9000, 60), np.full(3, 200)]
    assert tiles(ql, ql, W.LOCAL, True) == {("roll_i32", 8), ("roll_i32", 16)}


@pytest.mark.parametrize("n,cols,mode,cigar,rolls", [(2100, 300, W.LOCAL, True, True),
                                                     (2100, 500, W.LOCAL, True, False),
                                                     (3072, 500, W.LOCAL, True, False),
                                                     (3073, 500, W.LOCAL, True, True),
                                                     (2100, 500, W.GLOBAL, True, True),
                                                     (2100, 500, W.EXTEND, True, True)])
def test_local_paths_against_long_references(n, cols, mode, cigar, rolls):
    got = tiles(np.full(n, 250), np.full(n, cols), mode, cigar)
    assert got == ({("roll_i32", 16)} if rolls else {("strip_i32", 8)})
