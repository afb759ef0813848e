"""The calls this library is measured on.

Each case is one batch, of a shape that a program using the library meets, run
through the public binding: the plan and the device buffers are made once, one
pass executes the plan on the batch.  listed() gives the fixed ones, draw()
more of the same ranges.  A case is a dict of plain values:

  op      nw (global, full matrix), sw (local, full matrix), band (global,
          static band), xdrop / zdrop (seed extension), search (score-major
          search), fold (RNA folding)
  n       pairs (xdrop / zdrop: seeds of two sides each; fold: sequences)
  lo, hi  shortest and longest reference (protein sw: median lo, longest hi)
  div     share of edited bases between query and reference (extensions draw
          theirs, 5 to 25%, side by side: div is their mean)
  cigar   whether the alignment paths come back too
  alphabet 4 (DNA) or 20 (protein); w, x: band half-width, drop threshold
"""
import functools
import math

import numpy as np
import torch

from paper_2607_06225_amd import aln
from paper_2607_06225_amd import workloads as W


def listed():
    return [
        # one small request: a handful of short amplicons, ragged, with paths;
        # the call's latency and launches
        dict(name="nw_small", op="nw", n=16, lo=60, hi=300, div=0.10, cigar=True, alphabet=4),
        # the 256 x 1 kbp global batch: pairwise alignment of contigs or genes
        dict(name="nw_dna_1k", op="nw", n=256, lo=1000, hi=1000, div=0.10, cigar=True, alphabet=4),
        # protein database search: scores and end cells, lognormal lengths
        dict(name="sw_protein", op="sw", n=16384, lo=350, hi=2000, div=0.60, cigar=False,
             alphabet=20),
        # short reads realigned to candidate windows, with paths
        dict(name="sw_reads", op="sw", n=8192, lo=150, hi=320, div=0.05, cigar=True, alphabet=4),
        # long-read overlaps of a few kbp in a narrow band, with paths
        dict(name="band_reads", op="band", n=2048, lo=1000, hi=9000, div=0.08, cigar=True,
             alphabet=4, w=64),
        # whole long reads, 10 to 100 kbp at 12% errors, in a wide band
        dict(name="band_long", op="band", n=384, lo=10000, hi=100000, div=0.12, cigar=True,
             alphabet=4, w=256),
        # seed extension, scores only (the mapping stage that filters seeds)
        dict(name="xdrop_ext", op="xdrop", n=50000, lo=150, hi=5000, div=0.15, cigar=False,
             alphabet=4, x=100),
        # seed extension with paths (the seeds that were kept)
        dict(name="xdrop_cigar", op="xdrop", n=12500, lo=150, hi=5000, div=0.15, cigar=True,
             alphabet=4, x=100),
        # the same extensions under the Z-drop rule
        dict(name="zdrop_ext", op="zdrop", n=12500, lo=150, hi=5000, div=0.15, cigar=False,
             alphabet=4, x=100),
        # edit distance of similar sequences by the score-major search
        dict(name="edit_search", op="search", n=4096, lo=2000, hi=2000, div=0.05, cigar=False,
             alphabet=4, affine=False),
        # the same under gap-affine penalties
        dict(name="affine_search", op="search", n=4096, lo=2000, hi=2000, div=0.05, cigar=False,
             alphabet=4, affine=True),
        # RNA folding without pruning, the span of RNA lengths of the experiment
        dict(name="rna_fold", op="fold", n=2048, lo=76, hi=500, x=-1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["nw", "nw", "sw_protein", "sw_reads", "band", "band", "xdrop", "xdrop_cigar",
                     "zdrop", "search", "affine", "fold"])
    if op == "nw":
        alphabet = rng.choice([4, 4, 20])
        hi = _log(rng, 40, 2500 if alphabet == 4 else 1000)
        n = min(_log(rng, 1, 4096), max(1, int(1.5e9 / (hi * hi))))
        return dict(op="nw", n=n, lo=max(1, int(hi * rng.uniform(0.3, 1.0))), hi=hi,
                    div=round(rng.uniform(0.01, 0.30), 3), cigar=rng.random() < 0.75,
                    alphabet=alphabet)
    if op == "sw_protein":
        return dict(op="sw", n=_log(rng, 3, 20000), lo=_log(rng, 100, 500), hi=2000,
                    div=round(rng.uniform(0.3, 0.8), 3), cigar=False, alphabet=20)
    if op == "sw_reads":
        lo = _log(rng, 50, 300)
        return dict(op="sw", n=_log(rng, 16, 8192), lo=lo, hi=lo + _log(rng, 10, 300),
                    div=round(rng.uniform(0.01, 0.15), 3), cigar=True,
                    alphabet=4)
    if op == "band":
        hi = _log(rng, 300, 50000)
        w = _log(rng, 8, 400)
        n = min(_log(rng, 1, 3000), max(1, int(6e9 / (hi * (2 * w + 1)))))
        return dict(op="band", n=n, lo=max(1, int(hi * rng.uniform(0.1, 1.0))), hi=hi,
                    div=round(rng.uniform(0.02, 0.15), 3), cigar=rng.random() < 0.75, alphabet=4,
                    w=w)
    if op in ("xdrop", "xdrop_cigar", "zdrop"):
        hi = _log(rng, 200, 6000)
        most = 50000 if op == "xdrop" else 12000
        n = min(_log(rng, 8, most), int(1e8 / hi))
        return dict(op=op.split("_")[0], n=n, lo=max(20, int(hi * rng.uniform(0.03, 0.9))), hi=hi,
                    div=0.15, cigar=op == "xdrop_cigar", alphabet=4,
                    x=rng.randint(30, 120))
    if op in ("search", "affine"):
        hi = _log(rng, 100, 2300 if op == "affine" else 8000)
        div = round(rng.uniform(0.01, 0.15), 3)
        n = min(_log(rng, 1, 4096), max(1, int(1.2e9 / (hi * hi) * 0.15 / div)))
        return dict(op="search", n=n, lo=max(1, int(hi * rng.uniform(0.5, 1.0))), hi=hi, div=div,
                    cigar=False, alphabet=4, affine=op == "affine")
    hi = _log(rng, 40, 511)
    return dict(op="fold", n=_log(rng, 1, 2048), lo=max(1, int(hi * rng.uniform(0.1, 1.0))), hi=hi,
                x=rng.choice([-1, -1, 2, 5]))


# ------------------------------------------------------------------- inputs
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


class _Draws:
    """Seeded draws on the device (the inputs of a case, made from its seed)."""

    def __init__(self, seed):
        self.dev = _device()
        self.gen = torch.Generator(device=self.dev).manual_seed(int(seed))

    def uniform(self, n):
        return torch.rand(int(n), generator=self.gen, device=self.dev)

    def normal(self, n):
        return torch.randn(int(n), generator=self.gen, device=self.dev)

    def integers(self, lo, hi, n):
        return torch.randint(int(lo), int(hi) + 1, (int(n),), generator=self.gen, device=self.dev)

    def codes(self, n, alphabet):
        return torch.randint(0, alphabet, (int(n),), generator=self.gen, device=self.dev,
                             dtype=torch.uint8)


def _starts(lengths):
    return torch.cumsum(lengths, 0) - lengths


def _each(lengths):
    """For every base of the concatenated segments, its place in its segment."""
    return torch.arange(int(lengths.sum()), device=lengths.device) - torch.repeat_interleave(
        _starts(lengths), lengths)


def _edited(d, L, div, alphabet, w_sub=2, w_ins=1, w_del=1):
    """References of lengths L and their edited copies, concatenated: codes
    and lengths of both.  An edit replaces a base, inserts one after it or
    drops it, with the given weights; div is one rate, or one a pair."""
    n = int(L.sum())
    ref = d.codes(n, alphabet)
    rate = torch.repeat_interleave(div, L) if torch.is_tensor(div) else div
    tot = w_sub + w_ins + w_del
    kind = d.uniform(n) / rate * tot  # >= tot: not edited
    cnt = torch.ones(n, dtype=torch.int64, device=d.dev)
    cnt[(kind >= w_sub) & (kind < w_sub + w_ins)] = 2
    cnt[(kind >= w_sub + w_ins) & (kind < tot)] = 0
    other = (ref + 1 + d.codes(n, alphabet - 1)) % alphabet
    q = torch.repeat_interleave(torch.where(kind < w_sub, other, ref), cnt)
    upto = torch.cumsum(cnt, 0)
    ins = upto[cnt == 2] - 1
    q[ins] = d.codes(ins.numel(), alphabet)
    ends = torch.cat([upto.new_zeros(1), upto])[torch.cat([L.new_zeros(1), torch.cumsum(L, 0)])]
    return q, torch.diff(ends), ref, L


def _flanked(d, x, lengths, before, after):
    """Every segment of x between that many random bases."""
    tot = before + lengths + after
    out = d.codes(int(tot.sum()), 4)
    out[torch.repeat_interleave(_starts(tot) + before, lengths) + _each(lengths)] = x
    return out, tot


def _host(x, dtype):
    return x.cpu().numpy().astype(dtype, copy=False)


def _batch(case, q, ql, r, rl, matrix, go, ge, mode, prune):
    return W.Batch(case["op"], _host(q, np.uint8), _host(_starts(ql), np.int64),
                   _host(ql, np.int32), _host(r, np.uint8), _host(_starts(rl), np.int64),
                   _host(rl, np.int32), matrix, go, ge, mode, prune, case.get("w", 0),
                   case.get("x", 0), bool(case["cigar"]))


def _inputs(case, seed):
    op, n, lo, hi = case["op"], case["n"], case["lo"], case["hi"]
    if op == "fold":
        return W.rna_fold(n=n, seed=seed, min_len=lo, max_len=hi, xdrop=case["x"])
    d = _Draws(seed)
    if op in ("xdrop", "zdrop"):
        # two sides a seed, each at its own divergence of 5 to 25%, then an
        # unrelated flank of a tenth of the length
        L = d.integers(lo, hi, 2 * n)
        q, ql, r, rl = _edited(d, L, 0.05 + 0.20 * d.uniform(2 * n), 4)
        none, flank = torch.zeros_like(L), (L + 9) // 10
        q, ql = _flanked(d, q, ql, none, flank)
        r, rl = _flanked(d, r, rl, none, flank)
        return _batch(case, q, ql, r, rl, W.dna_matrix(2, -4), -4, -2, W.EXTEND,
                      W.ZDROP if op == "zdrop" else W.XDROP)
    if op == "sw" and case["alphabet"] == 20:
        # lognormal lengths around lo; three in ten queries share a window with
        # their reference, div of whose residues differ
        ql, rl = (torch.clamp(torch.round(lo * torch.exp(0.6 * d.normal(n))), 50, hi).long()
                  for _ in range(2))
        q, r = d.codes(int(ql.sum()), 20), d.codes(int(rl.sum()), 20)
        win = torch.where(d.uniform(n) < 0.3, torch.minimum(ql, rl), torch.zeros_like(ql))
        at, keep = _each(win), d.uniform(int(win.sum())) >= case["div"]
        src = torch.repeat_interleave(_starts(rl), win) + at
        dst = torch.repeat_interleave(_starts(ql), win) + at
        q[dst[keep]] = r[src[keep]]
        return _batch(case, q, ql, r, rl, W.protein_matrix(202), -11, -1, W.LOCAL, W.FULL)
    if op == "sw":
        # reads of about lo bases, each from somewhere inside a window of about
        # hi bases at most
        q, ql, r, rl = _edited(d, torch.full((n,), lo, dtype=torch.int64, device=d.dev),
                               case["div"], 4)
        most = max(0, (hi - lo) // 2)
        r, rl = _flanked(d, r, rl, d.integers(0, most, n), d.integers(0, most, n))
        return _batch(case, q, ql, r, rl, W.dna_matrix(2, -4), -4, -2, W.LOCAL, W.FULL)
    L = d.integers(lo, hi, n)
    if op == "band":
        q, ql, r, rl = _edited(d, L, case["div"], 4, 3, 5, 4)
        return _batch(case, q, ql, r, rl, W.dna_matrix(1, -2), -2, -1, W.GLOBAL, W.BAND)
    q, ql, r, rl = _edited(d, L, case["div"], case["alphabet"])
    if op == "search":
        m, go, ge = (W.dna_matrix(0, -4), -6, -2) if case["affine"] else (W.dna_matrix(0, -1), 0, -1)
        return _batch(case, q, ql, r, rl, m, go, ge, W.GLOBAL, W.SEARCH)
    if case["alphabet"] == 20:
        return _batch(case, q, ql, r, rl, W.protein_matrix(202), -11, -1, W.GLOBAL, W.FULL)
    return _batch(case, q, ql, r, rl, W.dna_matrix(2, -4), -4, -2, W.GLOBAL, W.FULL)


# -------------------------------------------------------------------- passes
@functools.lru_cache(maxsize=None)
def _context():
    return aln.Context(0)


@functools.lru_cache(maxsize=None)
def _scoring(matrix, alphabet, gap_open, gap_extend):
    m = np.frombuffer(matrix, dtype=np.int32).reshape(alphabet, alphabet)
    return _context().set_scoring(m, gap_open, gap_extend)


def prepare(case, seed):
    ctx = _context()
    b = _inputs(case, seed)
    if case["op"] == "fold":
        plan = aln.fold_plan(ctx, b)
        ws = torch.empty(max(plan.workspace_bytes, 1), dtype=torch.uint8, device="cuda")
        res = torch.zeros(b.n * aln.FOLD_RESULT_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
        words = res.view(torch.int32).view(b.n, -1)
        return dict(fold=True, ctx=ctx, plan=plan, batch=aln.FoldDeviceBatch(b), ws=ws, res=res,
                    out={"score": words[:, 0], "result": words})
    sid = _scoring(np.ascontiguousarray(b.matrix, dtype=np.int32).tobytes(), b.alphabet,
                   b.gap_open, b.gap_extend)
    plan = ctx.plan(sid, b.q_len, b.r_len, b.mode, b.prune, b.band_w, b.xdrop,
                    want_cigar=b.want_cigar)
    buf = aln.Buffers(plan)
    words = buf.res.view(torch.int32).view(b.n, -1)
    out = {"score": words[:, 0], "result": words}
    if b.want_cigar:
        # room for any lengths of the case, as a program that reuses one buffer
        # over many batches has it
        buf.cigar = torch.zeros(max(plan.cigar_words, b.n * int(2.6 * case["hi"] + 64)),
                                dtype=torch.int32, device="cuda")
        out["cigar"] = buf.cigar
    return dict(fold=False, ctx=ctx, plan=plan, batch=aln.DeviceBatch(b), buf=buf, out=out)


def run(s):
    if s["fold"]:
        aln.fold_execute(s["ctx"], s["plan"], s["batch"], s["ws"], s["res"])
    else:
        buf = s["buf"]
        s["ctx"].execute(s["plan"], s["batch"], buf.ws, buf.res, buf.cigar)
    return s["out"]


def work(case):
    """Codes in, results and path words out; the integer operations of the
    recurrence's cells (8 global, 10 local or X-drop, 12 Z-drop; folding: 2 a
    bifurcation term; search: 7 a furthest-row entry)."""
    n, lo, hi = case["n"], case["lo"], case["hi"]
    if case["op"] == "fold":
        mean3 = sum(v ** 3 for v in (lo, (lo + hi) / 2, hi)) / 3
        return {"bytes": n * ((lo + hi) / 2 + 16 + 40), "flops": n * mean3 / 6 * 2}
    L = (lo + hi) / 2
    sides = 1
    if case["op"] == "sw" and case["alphabet"] == 20:
        m = min(lo * 1.2, hi)
        codes, ops = 2 * m, m * m * 10
    elif case["op"] == "sw":
        codes, ops = lo + (lo + hi) / 2, lo * (lo + hi) / 2 * 10
    elif case["op"] == "nw":
        codes, ops = 2 * L, L * L * 8
    elif case["op"] == "band":
        codes, ops = 2 * L, L * min(2 * case["w"] + 1, L) * 8
    elif case["op"] == "search":
        # the penalty grows by about 1 (unit) or 5.7 (affine) an edit
        s = case["div"] * L * (5.7 if case["affine"] else 1.0)
        codes, ops = 2 * L, s * s * (0.5 if case["affine"] else 1.0) * 7
    else:
        # the region kept around the best diagonal is about 0.4 X (X-drop) or
        # 0.7 Z (Z-drop) cells wide on each of about 2 L antidiagonals
        sides = 2
        wide = case["x"] * (0.7 if case["op"] == "zdrop" else 0.4)
        codes, ops = 2.2 * L, 2 * L * wide * (12 if case["op"] == "zdrop" else 10)
    words = 2 * case["div"] * L if case["cigar"] else 0
    return {"bytes": n * sides * (codes + 24 + 48 + 4 * words), "flops": n * sides * ops}


def exact(case, seed):
    """Scores of the full-matrix global and local alignments, by the plain
    recurrence in 64 bits, row by row over all pairs at once."""
    if case["op"] not in ("nw", "sw"):
        return None
    L = case["lo"] * 1.5 if case["alphabet"] == 20 and case["op"] == "sw" else case["hi"]
    if case["n"] * L * L > 3e8:
        return None
    b = _inputs(case, seed)
    n, M, N = b.n, int(b.q_len.max(initial=0)), int(b.r_len.max(initial=0))
    local, o, e, low = b.mode == W.LOCAL, b.gap_open, b.gap_extend, -(1 << 40)
    q, r = np.zeros((n, M), np.int64), np.zeros((n, N), np.int64)
    for p in range(n):
        q[p, :b.q_len[p]], r[p, :b.r_len[p]] = b.pair(p)
    cols = np.arange(N + 1)
    inside = cols[None, :] <= b.r_len[:, None]
    H = np.where(cols > 0, 0 if local else o + e * cols, 0) * np.ones((n, 1), np.int64)
    F = np.full((n, N + 1), low, np.int64)
    score = np.zeros(n, np.int64) if local else H[np.arange(n), b.r_len].copy()
    m = b.matrix.astype(np.int64)
    for i in range(1, M + 1):
        F = np.maximum(F + e, H + o + e)
        D = np.full((n, N + 1), low, np.int64)
        D[:, 1:] = H[:, :-1] + m[q[:, i - 1][:, None], r]
        D[:, 0] = 0 if local else o + e * i
        T = np.maximum(D, F)
        if local:
            T = np.maximum(T, 0)
        # E(i, j) = max over k < j of T(i, k) + o + (j - k) e
        E = np.full((n, N + 1), low, np.int64)
        E[:, 1:] = np.maximum.accumulate(T - e * cols, axis=1)[:, :-1] + o + e * cols[1:]
        H = np.maximum(T, E)
        here = i <= b.q_len
        if local:
            best = np.where(inside, H, 0).max(axis=1)
            score = np.where(here, np.maximum(score, best), score)
        else:
            score = np.where(i == b.q_len, H[np.arange(n), b.r_len], score)
    return {"score": score.astype(np.int32), "result": None, "cigar": None}
