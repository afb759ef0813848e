// kernels_roll.hip -- Gotoh H/E/F with traceback on gfx950 for narrow bands and
// short pairs: row blocks that roll around a group of lanes (int32 scores).
//
// Schedule.  Block b is the R query rows bR + 1 .. bR + R.  A group of LG lanes
// (16, four pairs per wavefront, or the whole wavefront) owns one pair; block b
// runs on lane b mod LG, one column behind block b - 1: at step t it is on
// column j = t - b.  The bottom row's (H + o + e, F) moves to the next lane by
// one rotating DPP each, so block LG follows block LG - 1 on lane 0 without a
// hand-over through memory.
//
//   Static band (half-width w).  A block is in its band for about 2w + R steps
//   and the lane's next block starts LG (1 + R N / M) steps after this one did:
//   when that is longer (roll_fits), a lane is through with a block before its
//   next one starts, and takes it up at a multiple of 8 steps.  A pair takes
//   about M (1 + 1/R) steps; a strip of 64 R rows (kernels_strip.hip) takes 2w +
//   64 R + 63, nearly all of them shift and skew where the band is narrow.
//
//   Full matrix, M <= LG R: the same with every row's band 1..N and one block
//   a lane.
//
// Cells outside a row's band, or outside 1..N, are evaluated and their H set to
// minus infinity; E and F need no mask (left of a band only F can be finite and
// it flows down into cells also left of the band, right of it only E, flowing
// right).  Column 0 takes its formula at the step its block passes it.  A block
// past its last column, or not yet at its first, hands minus infinity down.
//
// Reference codes come from an LDS ring, one unaligned 8-byte read a lane and 8
// steps; the query's next rows from another when a lane takes up a block.  Both
// are refilled 64 codes at a time from registers loaded one refill before.
//
// Codes (4 bits a cell, as kernels_strip.hip's band strips): block b keeps Lw =
// roll_code_steps() steps from u_b, its first in-band step rounded down to
// roll_code_align(R), at (b Lw + t - u_b) R / 2; eight steps are R words, word r
// row r's nibbles, the earlier step higher.
#include "internal.h"

#include <type_traits>

namespace alnk {

namespace {

constexpr int kRollRing = 256; // codes per ring, and bytes repeated after it
constexpr int kRollMirror = 16;
constexpr int kRollGroup = 2 * (kRollRing + kRollMirror); // LDS bytes of one pair

// v = 2v + bit, a lane's bit taken from a mask of the wavefront as the carry.
// (Masks are combined and kept as such: a bool kept over a step, or built of
// two compares, costs a select and another compare.)
__device__ __forceinline__ void roll_shift_in(uint32_t &v, unsigned long long m) {
  unsigned long long cc;
  asm("v_addc_co_u32_e64 %0, %1, %2, %2, %3" : "=v"(v), "=s"(cc) : "v"(v), "s"(m));
  (void)cc;
}
__device__ __forceinline__ unsigned long long lanes_of(bool b) { return __builtin_amdgcn_ballot_w64(b); }

// lane l of a group reads lane l - 1, its first lane the last one's
template <int LG> __device__ __forceinline__ int rotate1(int v) {
  return LG == 64 ? __builtin_amdgcn_mov_dpp(v, 0x13C, 0xf, 0xf, true)  // wave_ror:1
                  : __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, true); // row_ror:1
}

} // namespace

template <int R, int LG, int MODE, bool TB, bool BAND>
__global__ __launch_bounds__(64) void roll_kernel(StripArgs a) {
  static_assert(LG == 16 || LG == 64, "a group is a DPP row or a wavefront");
  constexpr int AL = roll_code_align(R);
  // LOCAL / EXTEND, full matrix: a row's best as one key, the score above 0xffff
  // - j (scores at most 127 * 256, N < 65536; EXTEND's of any size below zero, and
  // a masked H, count as score 0, which is no result)
  constexpr bool KEY = !BAND && MODE != ALN_GLOBAL;
  __shared__ __align__(16) uint8_t smem[(64 / LG) * kRollGroup];
  const int lane = threadIdx.x;
  const int gl = lane & (LG - 1);
  uint8_t *rring = smem + (lane / LG) * kRollGroup;
  uint8_t *qring = rring + kRollRing + kRollMirror;
  const int task = blockIdx.x * (64 / LG) + lane / LG;
  const bool have = task < a.ntasks;
  const PairTask tk = a.tasks[have ? task : 0];
  const int p = tk.pair;
  const int M = a.b.q_len[p], N = a.b.r_len[p];
  const uint8_t *Q = a.b.q + a.b.q_off[p];
  const uint8_t *Rs = a.b.r + a.b.r_off[p];
  const DevScoring *sc = a.sc;
  const int go = sc->gap_open, ge = sc->gap_extend, goe = go + ge;
  const int w = a.band_w;
  const bool run = have && M > 0 && N > 0;
  const int nblocks = run ? (M + R - 1) / R : 0;
  uint32_t tab[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) tab[c] = c < sc->alphabet ? sc->rowtab[c] : 0x80808080u;
  auto row_scores = [&](int c) { // scores of query code c against codes 0..3
    const uint32_t x = (c & 1) ? tab[1] : tab[0], y = (c & 1) ? tab[3] : tab[2];
    return (c & 2) ? y : x;
  };

  // rings: codes 64n .. 64n + 63 at a time, 64 / LG per lane; reference codes
  // as bit offsets into a row's scores
  constexpr int SB = 64 / LG;
  auto fetch = [&](const uint8_t *src, int len, int top) { // codes top + SB gl ..
    uint32_t v = 0;
#pragma unroll
    for (int k = 0; k < SB; ++k) {
      const int at = top + SB * gl + k;
      const uint32_t c = run ? (uint32_t)src[min(at, len - 1)] & 3u : 0u;
      v |= c << (8 * k);
    }
    return v;
  };
  auto put = [&](uint8_t *ring, int top, uint32_t v) {
    const int at = (top + SB * gl) & (kRollRing - 1);
    if constexpr (SB == 1) {
      ring[at] = (uint8_t)v;
      if (at < kRollMirror) ring[kRollRing + at] = (uint8_t)v;
    } else {
      *reinterpret_cast<uint32_t *>(ring + at) = v;
      if (at < kRollMirror) *reinterpret_cast<uint32_t *>(ring + kRollRing + at) = v;
    }
  };

  // ---- the lane's block
  int b = gl;
  int Hl[R], EN[R], rb[R], rj[R], bb[R], wd[R], B[R];
  uint32_t rowtab[R];
  unsigned long long eo[R]; // lanes whose next E opens from H
  // band centre floor(iN/M) of the block's first row, with its remainder;
  // steps of one row and of LG R rows
  const int q1 = run ? N / M : 0, r1 = run ? N - q1 * M : 0;
  const int64_t blkN = (int64_t)LG * R * N;
  const int qs = run ? (int)(blkN / M) : 0, rs = run ? (int)(blkN - (int64_t)qs * M) : 0;
  int cen = 0, rem = 0;
  if (run) {
    const int64_t x = ((int64_t)b * R + 1) * N;
    cen = (int)(x / M);
    rem = (int)(x - (int64_t)cen * M);
  }
  const int Lw = roll_code_steps(max(M, 1), N, w, R);
  int u_b = 0, t_done = 0; // window start; the step from which the lane may leave the block
  uint8_t *tbl = nullptr;
  int64_t ncells = 0;
  // rows of block b: scores (from the query code fetched by `code`), band as steps
  auto take_block = [&](auto code) {
    int c = cen, m = rem;
    u_b = (max(1, cen - w) + b) & ~(AL - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = b * R + 1 + r;
      const bool valid = i <= M && b < nblocks;
      const int lo = BAND ? max(1, c - w) : 1, hi = BAND ? min(N, c + w) : N;
      const bool some = valid && hi >= lo;
      bb[r] = some ? lo + b : 1 << 30; // t - bb wraps above every width
      wd[r] = some ? hi - lo : 0;
      ncells += some ? hi - lo + 1 : 0;
      if (BAND && r == R - 1) t_done = roll_leave(hi + b, R);
      rowtab[r] = valid ? row_scores(code(i - 1)) : 0x80808080u;
      if (BAND) {
        c += q1;
        m += r1;
        if (m >= M) {
          m -= M;
          c += 1;
        }
      }
      Hl[r] = NEG32;
      EN[r] = NEG32;
      rb[r] = 0;
      rj[r] = 0;
    }
    if (TB) tbl = a.tb + tk.tb_off + (size_t)b * Lw * (R / 2);
  };
#pragma unroll
  for (int r = 0; r < R; ++r) eo[r] = ~0ull;
  take_block([&](int i) { return run ? (int)Q[min(i, M - 1)] & 3 : 0; });
  {
    int c = cen, m = rem;
#pragma unroll
    for (int r = 0; r < R; ++r) { // column 0 where it lies in the band
      const int i = b * R + 1 + r;
      B[r] = (!BAND || c <= w) ? (MODE == ALN_LOCAL ? 0 : go + i * ge) : NEG32;
      c += q1;
      m += r1;
      if (m >= M) {
        m -= M;
        c += 1;
      }
    }
  }
  // rings: reference columns 1..64 and the next 64 in flight; query rows after
  // the first LG blocks
  int rtop = 0, qtop = LG * R, bmin = 0;
  put(rring, 0, fetch(Rs, N, 0) * 8u);
  rtop = 64;
  uint32_t rnext = fetch(Rs, N, rtop), qnext = 0;
  if (BAND) {
    put(qring, qtop, fetch(Q, M, qtop));
    qtop += 64;
    qnext = fetch(Q, M, qtop);
  }

  int out_t = NEG32 + goe, out_f = NEG32, hd_top = NEG32;
  int best = 0, best_i = 0, best_j = 0;
  auto fold_best = [&] { // the block's best cell: rows in order, so strictly greater
    if (MODE == ALN_GLOBAL) return;
#pragma unroll
    for (int r = 0; r < R; ++r)
    {
      const int v = KEY ? rb[r] >> 16 : rb[r];
      if (v > best && b * R + 1 + r <= M) {
        best = v;
        best_i = b * R + 1 + r;
        best_j = KEY ? 0xffff - (rb[r] & 0xffff) : rj[r];
      }
    }
  };
  // GLOBAL: H(M, N) at the step its block is on column N
  const int bM = nblocks - 1, rM = run ? (M - 1) - bM * R : 0;
  const int t_end = run ? N + bM : -1;
  int gh = NEG32;
  const int t_stop = run ? (t_end & ~(AL - 1)) + AL : 0; // row M ends on column N, the last to
  int t_all = t_stop, n_min = run ? N : 0x7fffffff;
  if (LG < 64) {
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
      t_all = max(t_all, __shfl_xor(t_all, o, 64));
      n_min = min(n_min, __shfl_xor(n_min, o, 64));
    }
  }
  t_all = __builtin_amdgcn_readfirstlane(t_all);
  n_min = __builtin_amdgcn_readfirstlane(n_min);

  uint32_t acc[R], pend[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = pend[r] = 0;
  uint32_t cw[2];          // this lane's codes of the 8 steps
  bool oldest = b == bmin; // the lane of the pair's oldest block

  // FEED: the oldest block may be block 0, under row 0; C0: a block may be on
  // column 0; MASK: cells outside 1..N or the band; GH: the steps that hold some
  // pair's t_end
  auto step = [&](auto feed_tag, auto c0_tag, auto mask_tag, auto gh_tag, const int t, const int k) {
    constexpr bool FEED = decltype(feed_tag)::value, C0 = decltype(c0_tag)::value;
    constexpr bool MASK = decltype(mask_tag)::value, GH = decltype(gh_tag)::value;
    int above = NEG32 + goe;
    if (FEED) { // H(0, t) + o + e where (0, t) lies in the band
      const int h0 = (BAND && t > w) ? NEG32 : ((MODE == ALN_LOCAL || t == 0) ? 0 : go + t * ge);
      above = (!BAND || bmin == 0) ? h0 + goe : above;
    }
    const int rt = rotate1<LG>(out_t), rf = rotate1<LG>(out_f);
    const int in_t = oldest ? above : rt, in_f = oldest ? NEG32 : rf;
    const int sh = (int)(cw[k >> 2] >> (8 * (k & 3))); // low 5 bits: 8 * code
    int tu = in_t, fu = in_f, hd = hd_top;
    const uint32_t jkey = (uint32_t)(0xffff + b - t) & 0xffffu;
    const bool in_all = !BAND && (unsigned)(t - bb[0]) <= (unsigned)wd[0];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int sv = __builtin_amdgcn_sbfe((int)rowtab[r], sh, 8);
      const int f = max(fu + ge, tu);
      int hdiag = hd + sv;
      if (MODE == ALN_LOCAL) hdiag = max(hdiag, 0); // a zero stops a path before the diagonal does
      int h = max(max(hdiag, EN[r]), f);
      if (MASK) h = (BAND ? (unsigned)(t - bb[r]) <= (unsigned)wd[r] : in_all) ? h : NEG32;
      if (C0) h = t == b ? B[r] : h;
      const int tt = h + goe;
      const int en = max(EN[r] + ge, tt);
      if (TB) {
        const unsigned long long nd = lanes_of(h != hdiag), ne = lanes_of(h != EN[r]);
        roll_shift_in(acc[r], nd);
        roll_shift_in(acc[r], MODE == ALN_LOCAL ? (nd & ne) | lanes_of(h == 0) : ne);
        roll_shift_in(acc[r], eo[r]);
        roll_shift_in(acc[r], lanes_of(f == tu));
        eo[r] = lanes_of(en == tt);
      }
      if (KEY) {
        const int hk = MODE == ALN_EXTEND ? max(h, 0) : h; // (the shift would drop a sign)
        rb[r] = max(rb[r], (int)(((uint32_t)hk << 16) | jkey));
      } else if (MODE != ALN_GLOBAL) {
        if (h > rb[r]) {
          rb[r] = h;
          rj[r] = t - b;
        }
      }
      hd = Hl[r];
      Hl[r] = h;
      EN[r] = en;
      tu = tt;
      fu = f;
    }
    hd_top = in_t - goe;
    out_t = tu;
    out_f = fu;
    if (GH) { // (a register picked by rM would go through memory)
      int v = NEG32;
#pragma unroll
      for (int r = 0; r < R; ++r) v = max(v, rM == r ? Hl[r] : NEG32);
      gh = (t == t_end && b == bM) ? v : gh;
    }
  };
  using Yes = std::integral_constant<bool, true>;
  using No = std::integral_constant<bool, false>;

  // band: steps with a cell of row 0 in the band, or a block on column 0 (no
  // block taken up later starts there, roll_fits, nor is one taken up before
  // step w + 1)
  const int t_feed = BAND ? max(LG, w + 1) : 0x7fffffff;
  for (int t8 = 0; t8 < t_all; t8 += 8) {
    if (BAND) { // lanes through with their block take up the next
      const bool done = b + LG < nblocks && t8 >= t_done;
      const unsigned long long dm = __ballot(done);
      if (dm) {
        // (the query's rows are staged: 64 at a time, at least 16 blocks ahead)
        if (done) {
          fold_best();
          b += LG;
          cen += qs;
          rem += rs;
          if (rem >= M) {
            rem -= M;
            cen += 1;
          }
          take_block([&](int i) { return (int)qring[i & (kRollRing - 1)]; });
          out_t = NEG32 + goe;
          out_f = NEG32;
          hd_top = NEG32;
        }
        bmin += LG == 64 ? (int)__builtin_popcountll(dm)
                         : (int)__builtin_popcount((uint32_t)(dm >> (lane & 48)) & 0xffffu);
        oldest = b == bmin;
        const bool needq = qtop < (bmin + LG + 16) * R && qtop < M + 64;
        if (__ballot(needq)) {
          if (needq) {
            put(qring, qtop, qnext);
            qtop += 64;
            qnext = fetch(Q, M, qtop);
          }
        }
      }
    }
    {
      const bool needr = rtop < t8 + 16 - bmin && rtop < N + 64;
      if (__ballot(needr)) {
        if (needr) {
          put(rring, rtop, rnext * 8u);
          rtop += 64;
          rnext = fetch(Rs, N, rtop);
        }
      }
    }
    __builtin_memcpy(cw, rring + ((t8 - b - 1) & (kRollRing - 1)), 8);
    const bool gh8 = MODE == ALN_GLOBAL && __ballot((unsigned)(t_end - t8) < 8u) != 0;
    if (!BAND) {
      if (t8 < LG) {
#pragma unroll
        for (int k = 0; k < 8; ++k) step(Yes{}, Yes{}, Yes{}, Yes{}, t8 + k, k);
      } else if (t8 + 7 <= n_min && !gh8) { // every lane on a column of 1..N
#pragma unroll
        for (int k = 0; k < 8; ++k) step(Yes{}, No{}, No{}, No{}, t8 + k, k);
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) step(Yes{}, No{}, Yes{}, Yes{}, t8 + k, k);
      }
    } else if (t8 < t_feed) {
#pragma unroll
      for (int k = 0; k < 8; ++k) step(Yes{}, Yes{}, Yes{}, Yes{}, t8 + k, k);
    } else if (gh8) {
#pragma unroll
      for (int k = 0; k < 8; ++k) step(No{}, No{}, Yes{}, Yes{}, t8 + k, k);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) step(No{}, No{}, Yes{}, No{}, t8 + k, k);
    }
    if (TB) { // the 8 steps' codes (R = 2: 16 bytes every other time)
      const int tp = t8 - u_b;
      const bool mine = (unsigned)tp < (unsigned)Lw && b < nblocks;
      if constexpr (R == 2) {
        if (mine && (tp & 8)) *reinterpret_cast<uint4 *>(tbl + tp - 8) = make_uint4(pend[0], pend[1], acc[0], acc[1]);
        pend[0] = acc[0];
        pend[1] = acc[1];
      } else {
        if (mine) {
          uint32_t *dst = reinterpret_cast<uint32_t *>(tbl + (size_t)tp * (R / 2));
          if constexpr (R % 4 == 0) {
#pragma unroll
            for (int v = 0; v < R / 4; ++v)
              reinterpret_cast<uint4 *>(dst)[v] = make_uint4(acc[4 * v], acc[4 * v + 1], acc[4 * v + 2], acc[4 * v + 3]);
          } else {
#pragma unroll
            for (int v = 0; v < R / 2; ++v)
              reinterpret_cast<uint2 *>(dst)[v] = make_uint2(acc[2 * v], acc[2 * v + 1]);
          }
        }
      }
    }
  }
  fold_best();

  // ---- the pair's result
  if (MODE != ALN_GLOBAL) { // highest score, then smallest i, then smallest j
#pragma unroll
    for (int o = 1; o < LG; o <<= 1) {
      const int s2 = __shfl_xor(best, o, 64), i2 = __shfl_xor(best_i, o, 64), j2 = __shfl_xor(best_j, o, 64);
      const bool take = s2 > best || (s2 == best && (i2 < best_i || (i2 == best_i && j2 < best_j)));
      best = take ? s2 : best;
      best_i = take ? i2 : best_i;
      best_j = take ? j2 : best_j;
    }
  } else {
#pragma unroll
    for (int o = 1; o < LG; o <<= 1) gh = max(gh, __shfl_xor(gh, o, 64));
  }
#pragma unroll
  for (int o = 1; o < LG; o <<= 1) ncells += __shfl_xor(ncells, o, 64);
  if (!have || gl != 0) return;
  aln_result *res = a.res + p;
  if (MODE == ALN_GLOBAL) {
    if (!run) res->score = (M + N == 0) ? 0 : go + (M + N) * ge;
    else if (gh <= NEG32 / 2) {
      res->score = INT32_MIN;
      set_status(res, ALN_R_UNREACHABLE);
    } else {
      res->score = gh;
    }
    res->q_end = M;
    res->r_end = N;
  } else {
    res->score = best;
    res->q_end = best_i;
    res->r_end = best_j;
  }
  res->cells = ncells;
}

namespace {

template <int R, int LG, bool BAND>
hipError_t launch_roll_t(int mode, bool tb, const StripArgs &a, hipStream_t s) {
  const dim3 grid((a.ntasks + 64 / LG - 1) / (64 / LG)), block(64);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, 0, s, a);
    return hipGetLastError();
  };
  switch (mode) {
  case ALN_GLOBAL: return tb ? go(roll_kernel<R, LG, ALN_GLOBAL, true, BAND>) : go(roll_kernel<R, LG, ALN_GLOBAL, false, BAND>);
  case ALN_LOCAL: return tb ? go(roll_kernel<R, LG, ALN_LOCAL, true, BAND>) : go(roll_kernel<R, LG, ALN_LOCAL, false, BAND>);
  case ALN_EXTEND: return tb ? go(roll_kernel<R, LG, ALN_EXTEND, true, BAND>) : go(roll_kernel<R, LG, ALN_EXTEND, false, BAND>);
  default: return hipErrorInvalidValue;
  }
}

} // namespace

// Narrow bands: 2 or 4 rows a block on 16 or 64 lanes; full matrix of up to 16
// R rows: 8, 10 or 16 rows a block on 16 lanes.
hipError_t launch_roll(int rows, int mode, bool tb, const StripArgs &a, hipStream_t s) {
  if (a.ntasks <= 0) return hipSuccess;
  if (a.roll_full) {
    if (a.roll_lanes != 16) return hipErrorInvalidValue;
    switch (rows) {
    case 8: return launch_roll_t<8, 16, false>(mode, tb, a, s);
    case 10: return launch_roll_t<10, 16, false>(mode, tb, a, s);
    case 16: return launch_roll_t<16, 16, false>(mode, tb, a, s);
    default: return hipErrorInvalidValue;
    }
  }
  if (rows == 2)
    return a.roll_lanes == 16 ? launch_roll_t<2, 16, true>(mode, tb, a, s) : launch_roll_t<2, 64, true>(mode, tb, a, s);
  if (rows == 4)
    return a.roll_lanes == 16 ? launch_roll_t<4, 16, true>(mode, tb, a, s) : launch_roll_t<4, 64, true>(mode, tb, a, s);
  return hipErrorInvalidValue;
}

} // namespace alnk
