"""Packed Smith-Waterman: last strips of 4 to 16 rows a lane on 16-lane groups, and wide
items (one pair, the strip's lower half in the high halves of the registers) over one and
several strips: whole numbers, equal to the oracle."""
import numpy as np
import pytest

from paper_2607_06225_amd import workloads as W
from tests.parity import compare, oracle_batch

pytestmark = pytest.mark.gpu

ROWS = [0, 1, 63, 64, 65, 127, 128, 129, 192, 193, 255, 256, 257, 320, 511, 512, 513, 769, 1023, 1024,
        1025, 1537, 2047, 2048, 2049, 2305, 4097]


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2607_06225_amd import aln
    assert torch.cuda.is_available()
    c = aln.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("tile", [4, 8, 12, 16])
@pytest.mark.parametrize("wide", [-1, 1])  # no wide items; every item wide
@pytest.mark.parametrize("letters,gap", [(20, (-11, -1)), (4, (0, -3)), (31, (-2, -2))])
def test_strips(ctx, tile, wide, letters, gap):
    from paper_2607_06225_amd import aln
    rng = np.random.default_rng(tile * 7 + wide + letters)
    qs, rs = [], []
    for M in ROWS:
        for N in (int(rng.integers(1, 20)), int(rng.integers(60, 200))):
            q = rng.integers(0, letters, size=M).astype(np.uint8)
            r = rng.integers(0, letters, size=N).astype(np.uint8)
            k = min(M, N) // 2  # a common stretch at the query's end: the best cell low down
            if k:
                r[N - k:] = q[M - k:]
            qs.append(q)
            rs.append(r)
    m = rng.integers(-4, 2, size=(letters, letters)).astype(np.int32)
    np.fill_diagonal(m, 5)
    b = W.pack_pairs(qs, rs, m, gap[0], gap[1], W.LOCAL, W.FULL, name=f"strips{tile}_{wide}_{letters}")
    print(f"[gpu] {b.name}", flush=True)
    ctx.set_tuning(dict(valid=True, sw16_rows=tile, sw16_wide_pct=wide, strip_rows=8))
    try:
        res, _ = aln.align(ctx, b)
        one, _ = aln.align(ctx, b, per_pair=True)
    finally:
        ctx.set_tuning(dict(valid=False))
    assert compare(b, res, None, oracle_batch(b)) == []
    assert np.array_equal(res, one)
