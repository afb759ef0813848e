"""The unpruned fold by 16 x 16 tiles: lengths on both sides of its tile edges and
of the number of workgroups a CU holds, every workgroup size, byte scores up to their
largest, pairs barred by any loop length; integers, so equal to the oracle."""
import numpy as np
import pytest

import oracle
from paper_2607_06225_amd import workloads as W

EDGES = [14, 15, 16, 17, 30, 31, 32, 33, 47, 48, 95, 96, 111, 112, 239, 240, 287, 288, 367, 368,
         383, 384, 495, 496, 507]


@pytest.fixture(scope="module")
def ctx():
    from paper_2607_06225_amd import aln
    c = aln.Context(0)
    yield c
    c.close()


def check(ctx, fb, block=0):
    from paper_2607_06225_amd import aln
    print(f"[gpu] fold {fb.name} n={fb.n} block={block}", flush=True)
    got = aln.fold(ctx, fb, block=block)
    exp = oracle.fold_batch(fb.pair, fb.x, fb.off, fb.length, min_loop=fb.min_loop, xdrop=fb.xdrop, nthreads=16)
    for k in ("score", "i", "j", "cells", "terms", "full", "status"):
        assert got[k].tolist() == exp[k].tolist(), k
    return got


def batch(lengths, pair, min_loop, seed):
    st = W.Stream(seed, 5)
    xs = [(st.u64(L) & np.uint64(3)).astype(np.uint8) for L in lengths]
    return W.pack_fold(xs, pair, name=f"tiles{seed}", min_loop=min_loop, xdrop=-1)


def weights(a, b, c):
    P = np.zeros((4, 4), dtype=np.int32)
    P[0, 3], P[3, 0], P[1, 2], P[2, 1], P[2, 3], P[3, 2] = a, a, b, b, c, c
    return P


@pytest.mark.gpu
@pytest.mark.parametrize("block", [256, 512, 1024])
@pytest.mark.parametrize("min_loop", [0, 3, 31, 2 ** 31 - 1])
def test_tile_edges(ctx, block, min_loop):
    check(ctx, batch(EDGES, W.rna_pair_table(), min_loop, 3 + block + min_loop % 97), block)


@pytest.mark.gpu
@pytest.mark.parametrize("top,longest", [(2, 253), (3, 169), (5, 101), (31, 17), (127, 3)])
def test_largest_byte_scores(ctx, top, longest):
    lengths = [longest, longest - 1, longest // 2, 1]
    fb = batch(lengths, weights(top, top - 1, 1), 0, 40 + top)
    check(ctx, fb)
    x = np.tile(np.array([0, 3], dtype=np.uint8), longest)[:longest]  # as many pairs as fit
    got = check(ctx, W.pack_fold([x], weights(top, 0, 0), name="full", min_loop=0, xdrop=-1))
    assert int(got["score"][0]) == top * (longest // 2)


@pytest.mark.parametrize("n,cus", [(40, 8), (700, 256), (3, 256)])
def test_two_launches_take_each_sequence_once(n, cus):
    from paper_2607_06225_amd import aln
    c = aln.Context.host(cus=cus)
    fb = W.rna_fold(n=n, seed=21, xdrop=-1)
    p = aln.fold_plan(c, fb)
    L, T = p.describe()
    assert len(L) <= 2
    assert sorted(T["pair"].tolist()) == list(range(fb.n))
    for t in T:
        assert L[int(t["launch"])]["tile"] >= int(fb.length[t["pair"]]) + 1
    p.close()
    c.close()
