"""Packed Smith-Waterman pairs without a reference (or a query) of every height and in every
kind of item, in a workspace that held other bytes: score 0 at (0, 0)."""
import numpy as np
import pytest
import torch

from paper_2607_06225_amd import aln, workloads as W
from tests.parity import compare, oracle_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("letters", [4, 20])
@pytest.mark.parametrize("n,rows,empty", [(3, (300, 300), 3), (8, (257, 2000), 8), (64, (100, 3000), 40),
                                          (4250, (200, 1000), 900), (9001, (250, 400), 3000)])
def test_empty_references(letters, n, rows, empty):
    assert torch.cuda.is_available()
    rng = np.random.default_rng(n + letters)
    qs = [rng.integers(0, letters, size=int(rng.integers(rows[0], rows[1] + 1))).astype(np.uint8)
          for _ in range(n)]
    rs = [np.zeros(0, np.uint8) if k < empty else qs[k][: 60 + k % 50].copy() for k in range(n)]
    if empty > 4:
        qs[1] = qs[1][:0]
        qs[-1] = qs[-1][:0]
    b = W.pack_pairs(qs, rs, np.where(np.eye(letters, dtype=bool), 3, -4).astype(np.int32), -5, -1,
                     W.LOCAL, W.FULL, name=f"empty{n}_{letters}")
    ctx = aln.Context(0)
    sid = ctx.set_scoring(b.matrix, b.gap_open, b.gap_extend)
    p = ctx.plan(sid, b.q_len, b.r_len, W.LOCAL, W.FULL)
    assert {l["family"] for l in p.describe()[0]} == {"sw16"}
    db, buf = aln.DeviceBatch(b), aln.Buffers(p)
    ores = oracle_batch(b)
    for per_pair in (False, True):
        if per_pair and n > 100:
            continue
        buf.ws.random_(0, 256)
        print(f"[gpu] {b.name} {per_pair}", flush=True)
        (ctx.execute_per_pair if per_pair else ctx.execute)(p, db, buf.ws, buf.res, None)
        torch.cuda.synchronize()
        assert compare(b, buf.results(n), None, ores) == []
    p.close()
    ctx.close()
