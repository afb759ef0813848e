// kernels_search.hip -- the score-major search schedule (Sec. 6.3) on
// gfx950: unit-cost edit distance, and gap-affine penalties (further below).
//
// The search transformation re-indexes the edit-distance recurrence by score:
// F(s, d) is the furthest row i reached on diagonal d = j - i with exactly s
// edits.  From F(s-1, .) three costly moves lead to diagonal d --
//   a mismatch   from (i, j) on d:     row F(s-1, d) + 1,
//   an insertion from (i, j) on d + 1: row F(s-1, d+1) + 1  (steps down),
//   a deletion   from (i, j) on d - 1: row F(s-1, d-1)      (steps right) --
// each kept only if it stays inside the matrix (row <= min(M, N - d)); the
// furthest survivor then advances for free along matching characters
// (extend).  The active diagonals widen by one on each side per score,
// clipped to the matrix: [max(-s, -M), min(s, N)].  The search stops at the
// first score s whose diagonal N - M reaches row M: s is the edit distance.
//
// One workgroup per pair, with both sequences and F (int16 per diagonal,
// -32768 for "not reached", so rows are at most 32767) in LDS.  Two forms:
// - search_group_kernel: 1 to 8 wavefronts and two F rows (previous score,
//   current score), used whenever both rows fit;
// - search_edit_kernel: one wavefront updating a single row in place, for
//   the longest pairs.  Lanes take 64 consecutive diagonals at a time; the
//   neighbours' old values come by DPP, the chunk's left neighbour from a
//   register saved before the previous chunk overwrote it, and its right
//   neighbour from LDS (not yet updated).
// Extension compares sixteen characters per step: of at most four symbols, packed two
// bits each, from two dwords of each sequence and a funnel shift; otherwise five aligned
// dword reads per sequence and four byte aligns, then the first differing byte.
// (Wide LDS reads at any alignment were slower than either: a lane at a time, they
// kept the LDS busy 73% of the time.)
//
// What bounds it: instructions, half of them scalar (loop, exec mask and row
// bookkeeping; 0.52 vector and 0.70 scalar a cycle and CU in the edit distance,
// 0.60 and 0.71 gap-affine), then the chain of one score: rows, first
// comparison, the path's further comparisons, barrier.  4 096 pairs of 2 000 nt at 5%:
// edit distance 249 -> 134 us (before: codes in bytes, four wavefronts always, rows of
// every diagonal),
// gap-affine (4, 6, 2) 3 364 -> 959 us (and every score, not the multiples of 2);
// 30 000 of 100..200 nt 129 -> 50 and 760 -> 157 us.
#include "internal.h"

namespace alnk {

// "Not reached": -32768 in the LDS row and, sign-extended, in registers.  A
// move from it stays negative (at most -32767) and every store maps a
// negative row back to -32768, so it never drifts towards a real row.
constexpr int16_t kNegF16 = -32768;
constexpr int kNegF = kNegF16;
constexpr int kSearchOutgrown = INT32_MIN; // a score that no pair has

__device__ __forceinline__ int fload(const int16_t *F, int idx) { return F[idx]; }

__device__ __forceinline__ int sdpp_shr1(int old, int v) { // lane l <- lane l-1
  return __builtin_amdgcn_update_dpp(old, v, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ int sdpp_shl1(int old, int v) { // lane l <- lane l+1
  return __builtin_amdgcn_update_dpp(old, v, 0x130, 0xf, 0xf, false);
}

// sixteen codes starting at byte `off` of an LDS sequence buffer (readable
// up to off + 19): five aligned dword reads and four byte aligns
__device__ __forceinline__ void load16(const uint8_t *buf, int off, uint64_t &lo, uint64_t &hi) {
  const uint32_t *w = reinterpret_cast<const uint32_t *>(buf + (off & ~3));
  const uint32_t sh = (uint32_t)(off & 3);
  const uint32_t w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3], w4 = w[4];
  lo = ((uint64_t)__builtin_amdgcn_alignbyte(w2, w1, sh) << 32) | __builtin_amdgcn_alignbyte(w1, w0, sh);
  hi = ((uint64_t)__builtin_amdgcn_alignbyte(w4, w3, sh) << 32) | __builtin_amdgcn_alignbyte(w3, w2, sh);
}

// advance row f of diagonal d while the next characters match, up to lim
// (sixteen characters per step: one LDS round trip and one loop test)
__device__ __forceinline__ int extend_bytes(const uint8_t *qs, const uint8_t *rs, int f, int d, int lim) {
  while (f < lim) {
    uint64_t qa, qb, ra, rb;
    load16(qs, f, qa, qb);
    load16(rs, f + d, ra, rb);
    const uint64_t x0 = qa ^ ra, x1 = qb ^ rb;
    const int n = x0 ? (__builtin_ctzll(x0) >> 3) : (x1 ? 8 + (__builtin_ctzll(x1) >> 3) : 16);
    f = min(f + n, lim);
    if (n < 16) break;
  }
  return f;
}

// The same with codes of two bits, sixteen a dword: two dwords of each sequence and a
// funnel shift are sixteen characters.  (Codes past a sequence's end may agree: lim
// stops there.)
__device__ __forceinline__ int extend_pairs(const uint32_t *qs, const uint32_t *rs, int f, int d,
                                            int lim) {
  for (;;) {
    const uint32_t *q = qs + (f >> 4), *r = rs + ((f + d) >> 4);
    const uint32_t x = __builtin_amdgcn_alignbit(q[1], q[0], 2 * f) ^
                       __builtin_amdgcn_alignbit(r[1], r[0], 2 * (f + d));
    const int n = (x ? __builtin_ctz(x) : 32) >> 1;
    f = min(f + n, lim);
    if (n < 16 || f >= lim) return f;
  }
}
template <bool PK>
__device__ __forceinline__ int extend(const uint8_t *qs, const uint8_t *rs, int f, int d, int lim) {
  if constexpr (PK)
    return extend_pairs(reinterpret_cast<const uint32_t *>(qs),
                        reinterpret_cast<const uint32_t *>(rs), f, d, lim);
  else
    return extend_bytes(qs, rs, f, d, lim);
}

// A sequence of len codes into LDS, four (sixteen) a thread from any address; only
// whole words inside the sequence are read as such.  Bytes: 20 bytes of padding after it.
__device__ __forceinline__ uint32_t word_of(const uint8_t *from, int k, int len, uint8_t pad) {
  uint32_t v = pad * 0x01010101u;
  if (k + 4 <= len)
    __builtin_memcpy(&v, from + k, 4);
  else
    for (int b = 0; b < 4; ++b)
      if (k + b < len) v = (v & ~(255u << (8 * b))) | ((uint32_t)from[k + b] << (8 * b));
  return v;
}
template <bool PK>
__device__ __forceinline__ void stage(uint8_t *to, const uint8_t *from, int len, uint8_t pad, int tid,
                                      int threads) {
  if constexpr (PK) {
    for (int k = tid; k < (len >> 4) + 2; k += threads) {
      uint32_t z = 0;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint32_t v = word_of(from, 16 * k + 4 * g, len, 0), t = v | (v >> 6);
        z |= ((t & 15u) | ((t >> 12) & 0xf0u)) << (8 * g);
      }
      reinterpret_cast<uint32_t *>(to)[k] = z;
    }
  } else {
    for (int k = 4 * tid; k < len + 20; k += 4 * threads) { // the buffer is whole words
      *reinterpret_cast<uint32_t *>(to + k) = word_of(from, k, len, pad);
    }
  }
}

// Entries of scores 0..S when e scores share a range of diagonals |d| <= score / e,
// clipped to -M..N.
__device__ __forceinline__ long long entries(int M, int N, int e, int S) {
  const int w = S / e;
  auto below = [](int lim, int w) -> long long { // sum of min(lim, k), k < w
    const long long m = min(lim, w - 1);
    return w <= 0 ? 0 : m * (m + 1) / 2 + (w - 1 - m) * lim;
  };
  const long long all = w + below(M, w) + below(N, w);
  return all * e + (long long)(S - w * e + 1) * (1 + min(M, w) + min(N, w));
}

template <bool PK>
__global__ __launch_bounds__(64) void search_edit_kernel(SearchArgs a) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int lane = threadIdx.x;
  const int task = blockIdx.x;
  if (task >= a.ntasks) return;
  const int p = __builtin_amdgcn_readfirstlane(a.tasks[task].pair);
  aln_result *res = a.res + p;
  if (__builtin_amdgcn_readfirstlane(res->status) != ALN_R_OK) return; // bad symbol
  const int M = __builtin_amdgcn_readfirstlane(a.b.q_len[p]);
  const int N = __builtin_amdgcn_readfirstlane(a.b.r_len[p]);
  const uint8_t *Q = a.b.q + a.b.q_off[p];
  const uint8_t *Rs = a.b.r + a.b.r_off[p];

  // LDS: query codes (M + 20 bytes, padding 0xFE), reference codes (N + 20,
  // padding 0xFF; the paddings never match each other or a code), F[d + M]
  uint8_t *qs = smem;
  uint8_t *rs = smem + a.lds_q;
  int16_t *F = reinterpret_cast<int16_t *>(smem + a.lds_q + a.lds_r);
  stage<PK>(qs, Q, M, 0xFE, lane, 64);
  stage<PK>(rs, Rs, N, 0xFF, lane, 64);
  for (int k = lane; k <= M + N; k += 64) F[k] = kNegF16;
  __syncthreads();

  const int dt = N - M; // the end cell's diagonal
  int s = 0, dmin = 0, dmax = 0;
  long long cells = 1;
  {
    const int f0 = extend<PK>(qs, rs, 0, 0, min(M, N));
    if (lane == 0) F[M] = (int16_t)f0;
  }
  __syncthreads();
  bool done = dt == 0 && __builtin_amdgcn_readfirstlane(fload(F, M)) >= M;
  while (!done && s < M + N) {
    ++s;
    dmin = max(dmin - 1, -M);
    dmax = min(dmax + 1, N);
    cells += dmax - dmin + 1;
    int carry = kNegF; // F(s-1, d0 - 1), saved before its chunk was overwritten
    for (int d0 = dmin; d0 <= dmax; d0 += 64) {
      const int d = d0 + lane;
      const bool act = d <= dmax;
      const int old = act ? fload(F, d + M) : kNegF;
      int right = sdpp_shl1(kNegF, old);
      int left = sdpp_shr1(kNegF, old);
      if (lane == 63) right = (d + 1 <= N) ? fload(F, d + 1 + M) : kNegF;
      if (lane == 0) left = carry;
      carry = __builtin_amdgcn_readlane(old, 63);
      const int lim = min(M, N - d);
      int f = kNegF;
      if (old + 1 <= lim) f = max(f, old + 1);     // mismatch
      if (right + 1 <= lim) f = max(f, right + 1); // insertion
      if (left <= lim) f = max(f, left);           // deletion
      if (act && f >= 0) f = extend<PK>(qs, rs, f, d, lim);
      if (act) F[d + M] = f >= 0 ? (int16_t)f : kNegF16;
    }
    done = dt >= dmin && dt <= dmax && __builtin_amdgcn_readfirstlane(fload(F, dt + M)) >= M;
  }
  if (lane == 0) {
    res->score = -s;
    res->q_end = M;
    res->r_end = N;
    res->cells = cells;
  }
}

// One to eight wavefronts per pair.  F(s-1, .) and F(s, .) live in two LDS rows
// that swap roles every score, so a step reads only the previous row and
// needs no carried neighbour: the active diagonals are cut into 64-diagonal
// chunks dealt round-robin to the wavefronts, and one barrier per score
// separates the writes of a score from the reads of the next.  A row entry
// outside the previous score's diagonals was never written (the active
// diagonals only widen, and each row is written on every other score), so it
// still reads "not reached".
// Rows first hold diagonals -dcap..dcap only where that lets more pairs share a CU; a
// pair whose range would leave them is marked by its score and left to a second
// launch with rows of every diagonal.  With LOOK (more than four symbols: unrelated pairs
// of four end within the cap, and the look's code takes 4% longer), so is one whose end
// cell's diagonal has, an eighth of the way to the cap, come forward too slowly to end
// within it: a pair that has to be searched twice costs the first search 1/64 of its
// entries, not all.  4 096 unrelated pairs of 2 000 letters of 20: 27.3 ms before, 12.8 with
// it (and four wavefronts a pair in the second launch); without capped rows 16.4.
template <int NWV, bool PK, bool LOOK>
__global__ __launch_bounds__(64 * NWV) void search_group_kernel(SearchArgs a) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int task = blockIdx.x;
  if (task >= a.ntasks) return;
  const int p = __builtin_amdgcn_readfirstlane(a.tasks[task].pair);
  aln_result *res = a.res + p;
  // the same status for every wavefront: the whole workgroup leaves
  if (__builtin_amdgcn_readfirstlane(res->status) != ALN_R_OK) return;
  const int M = __builtin_amdgcn_readfirstlane(a.b.q_len[p]);
  const int N = __builtin_amdgcn_readfirstlane(a.b.r_len[p]);
  const uint8_t *Q = a.b.q + a.b.q_off[p];
  const uint8_t *Rs = a.b.r + a.b.r_off[p];

  if (a.pass == 1 && __builtin_amdgcn_readfirstlane(res->score) != kSearchOutgrown) return;
  const bool capped = a.dcap > 0;
  const int off = capped ? a.dcap : M;              // row index of diagonal 0
  const int lo_st = capped ? max(-M, -a.dcap) : -M; // stored diagonals lo_st..hi_st
  const int hi_st = capped ? min(N, a.dcap) : N;

  uint8_t *qs = smem;
  uint8_t *rs = smem + a.lds_q;
  int16_t *Fp = reinterpret_cast<int16_t *>(smem + a.lds_q + a.lds_r);
  int16_t *Fn = reinterpret_cast<int16_t *>(smem + a.lds_q + a.lds_r + a.lds_f);
  stage<PK>(qs, Q, M, 0xFE, tid, 64 * NWV);
  stage<PK>(rs, Rs, N, 0xFF, tid, 64 * NWV);
  for (int k = 8 * tid; k < a.lds_f / 2; k += 8 * 64 * NWV) { // rows are whole 16 bytes
    *reinterpret_cast<uint4 *>(Fp + k) = make_uint4(0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u);
    *reinterpret_cast<uint4 *>(Fn + k) = make_uint4(0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u);
  }
  __syncthreads();
  if (tid == 0) Fp[off] = (int16_t)extend<PK>(qs, rs, 0, 0, min(M, N));
  __syncthreads();

  const int dt = N - M;
  const bool ends = dt >= lo_st && dt <= hi_st; // the end cell's diagonal is stored
  int s = 0, dmin = 0, dmax = 0;
  bool outgrown = false;
  // LOOK: the diagonals at which the pair's course is looked at
  const int look = a.dcap >> 3;
  int lo_lim = LOOK ? max(lo_st, -look) : lo_st, hi_lim = LOOK ? min(hi_st, look) : hi_st;
  for (;;) {
    // is the end cell reached at score s?  Known once score s + 1 is computed, whose
    // reads need not wait for it.
    int end = kNegF;
    if (ends) end = fload(Fp, dt + off);
    const int nmin = max(dmin - 1, -M), nmax = min(dmax + 1, N);
    const bool edge = nmin == lo_st || nmax == hi_st;
    outgrown = nmin < lo_lim || nmax > hi_lim; // only with capped rows (uniform)
    for (int d0 = outgrown ? nmax + 1 : nmin + 64 * wave; d0 <= nmax; d0 += 64 * NWV) {
      const int d = d0 + lane;
      if (d <= nmax) {
        const int16_t *src = Fp + d + off;
        const int old = src[0];
        int left, right;
        if (!edge) {
          left = src[-1];
          right = src[1];
        } else {
          left = d > lo_st ? src[-1] : kNegF;
          right = d < hi_st ? src[1] : kNegF;
        }
        // a row past the diagonal's end stands for the end, which was reached before:
        // every active diagonal has a row, the furthest of s edits at most
        const int lim = min(M, N - d);
        const int f = min(max(left, max(old, right) + 1), lim);
        Fn[d + off] = (int16_t)extend<PK>(qs, rs, f, d, lim);
      }
    }
    if (__builtin_amdgcn_readfirstlane(end) >= M || s >= M + N) {
      outgrown = false;
      break;
    }
    if (outgrown) {
      if (!LOOK || nmin < lo_st || nmax > hi_st) break;
      // (row M at this rate after M s / end edits, or an eighth more; a diagonal that s
      // edits have just reached says nothing)
      if (2 * abs(dt) <= look && M * s > __builtin_amdgcn_readfirstlane(end) * (a.dcap - a.dcap / 8)) break;
      lo_lim = lo_st;
      hi_lim = hi_st;
      continue; // (nothing of this score has been written)
    }
    __syncthreads();
    ++s;
    dmin = nmin;
    dmax = nmax;
    int16_t *t = Fp;
    Fp = Fn;
    Fn = t;
  }
  if (tid == 0 && outgrown) {
    res->score = kSearchOutgrown;
  } else if (tid == 0) {
    res->score = -s;
    res->q_end = M;
    res->r_end = N;
    res->cells = entries(M, N, 1, s);
  }
}

// Gap-affine penalties: mismatch x > 0, a gap of length L costs o + L e
// (o >= 0, e > 0), a match 0.  The search keeps three wavefronts per score,
// furthest rows as before:
//   E(s, d) = max(H(s-o-e, d-1), E(s-e, d-1))       a step right, same row
//   F(s, d) = max(H(s-o-e, d+1), F(s-e, d+1)) + 1   a step down
//   H(s, d) = max(H(s-x, d) + 1, E(s, d), F(s, d)), then extended along
//             matches,
// each candidate kept only if its source was reached and it stays inside the
// matrix (row <= min(M, N - d)).  A path of penalty s spends at least e per
// diagonal it moves, so the active diagonals are |d| <= s / e, clipped to the
// matrix.  The search stops at the first s with H(s, N - M) = M: s is the
// smallest penalty, minus the Gotoh global score under (0, -x, -o, -e).
// Every penalty is a multiple of g = gcd(x, o + e, e), and so is every score that is
// reached: the search counts in units of g, and the scores between, whose rows would all
// read "not reached", only add their diagonals to the count of entries.
// Rows for past scores live in LDS rings (H: ring_h rows, E and F: ring_e
// rows each, slot s mod ring size); the wavefronts share a pair as in
// search_group_kernel, one barrier per score.  A slot's earlier scores had
// narrower diagonal ranges, all rewritten when it is reused, so an entry
// outside a row's range still reads "not reached".
// Rows first hold diagonals -dcap..dcap only, so that several pairs share a
// CU; a pair whose range would leave them is flagged and recomputed by a
// second launch with rows of every diagonal.  A source diagonal outside the
// stored ones was never active (the range at an earlier score was inside
// them), so it reads "not reached".
template <int NWV, bool PK>
__global__ __launch_bounds__(64 * NWV) void search_affine_kernel(SearchArgs a) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int task = blockIdx.x;
  if (task >= a.ntasks) return;
  const int p = __builtin_amdgcn_readfirstlane(a.tasks[task].pair);
  aln_result *res = a.res + p;
  if (__builtin_amdgcn_readfirstlane(res->status) != ALN_R_OK) return;
  const int M = __builtin_amdgcn_readfirstlane(a.b.q_len[p]);
  const int N = __builtin_amdgcn_readfirstlane(a.b.r_len[p]);
  const uint8_t *Q = a.b.q + a.b.q_off[p];
  const uint8_t *Rs = a.b.r + a.b.r_off[p];
  if (a.pass == 1 && !(__builtin_amdgcn_readfirstlane(res->flags) & ALN_F_WIDENED)) return;
  const int X = a.pen_x, O = a.pen_o, E = a.pen_e; // in units of a.pen_g
  const bool capped = a.dcap > 0;
  const int off = capped ? a.dcap : M;             // row index of diagonal 0
  const int lo_st = capped ? max(-M, -a.dcap) : -M; // stored diagonals lo_st..hi_st
  const int hi_st = capped ? min(N, a.dcap) : N;

  uint8_t *qs = smem;
  uint8_t *rs = smem + a.lds_q;
  const int stride = a.lds_f; // bytes per row
  const int wrap_h = a.ring_h * stride, wrap_e = a.ring_e * stride;
  uint8_t *hring = smem + a.lds_q + a.lds_r;
  uint8_t *ering = hring + wrap_h, *fring = ering + wrap_e;
  stage<PK>(qs, Q, M, 0xFE, tid, 64 * NWV);
  stage<PK>(rs, Rs, N, 0xFF, tid, 64 * NWV);
  for (int k = 16 * tid; k < wrap_h + 2 * wrap_e; k += 16 * 64 * NWV) // rows are whole 16 bytes
    *reinterpret_cast<uint4 *>(hring + k) = make_uint4(0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u);
  __syncthreads();
  if (tid == 0) reinterpret_cast<int16_t *>(hring)[off] = (int16_t)extend<PK>(qs, rs, 0, 0, min(M, N));
  __syncthreads();

  const int dt = N - M;
  const bool ends = dt >= lo_st && dt <= hi_st; // the end cell's diagonal is stored
  const int smax = 2 * O + E * (M + N); // a gap of the whole query, then one of the reference
  // Rows by byte offset, kept incrementally: of this score, of the score before, and of
  // s - X, s - O - E, s - E (slots not yet written read "not reached").
  auto next = [](int o, int stride, int wrap) { return o + stride == wrap ? 0 : o + stride; };
  int s = 0;
  int hn = 0, hx = (a.ring_h - X) * stride, ho = (a.ring_h - O - E) * stride;
  int en = 0, ee = (a.ring_e - E) * stride;
  int w = 0, wr = 0; // s / E, s mod E
  bool outgrown = false;
  for (;;) {
    // is the end cell reached at score s?  Known once score s + 1 is computed, whose
    // reads need not wait for it.
    int end = kNegF;
    if (ends) end = fload(reinterpret_cast<const int16_t *>(hring + hn), dt + off);
    if (++wr == E) {
      wr = 0;
      ++w;
    }
    hn = next(hn, stride, wrap_h);
    hx = next(hx, stride, wrap_h);
    ho = next(ho, stride, wrap_h);
    en = next(en, stride, wrap_e);
    ee = next(ee, stride, wrap_e);
    const int dmin = max(-M, -w), dmax = min(N, w);
    outgrown = dmin < lo_st || dmax > hi_st; // only with capped rows (uniform)
    if (!outgrown) {
      const int16_t *Hx = reinterpret_cast<const int16_t *>(hring + hx) + off;
      const int16_t *Ho = reinterpret_cast<const int16_t *>(hring + ho) + off;
      const int16_t *Ee = reinterpret_cast<const int16_t *>(ering + ee) + off;
      const int16_t *Fe = reinterpret_cast<const int16_t *>(fring + ee) + off;
      int16_t *Hn = reinterpret_cast<int16_t *>(hring + hn) + off;
      int16_t *En = reinterpret_cast<int16_t *>(ering + en) + off;
      int16_t *Fn = reinterpret_cast<int16_t *>(fring + en) + off;
      const bool edge = dmin == lo_st || dmax == hi_st;
      for (int d0 = dmin + 64 * wave; d0 <= dmax; d0 += 64 * NWV) {
        const int d = d0 + lane;
        if (d <= dmax) {
          const int lim = min(M, N - d);
          int ev, fv, hv = Hx[d];
          if (!edge) {
            ev = max(Ho[d - 1], Ee[d - 1]); // a step right from diagonal d - 1
            fv = max(Ho[d + 1], Fe[d + 1]); // a step down from diagonal d + 1
          } else {
            ev = d > lo_st ? max(Ho[d - 1], Ee[d - 1]) : kNegF16;
            fv = d < hi_st ? max(Ho[d + 1], Fe[d + 1]) : kNegF16;
          }
          ev = ev <= lim ? ev : kNegF;
          fv = fv >= 0 && fv < lim ? fv + 1 : kNegF;
          hv = hv >= 0 && hv < lim ? hv + 1 : kNegF; // a mismatch on diagonal d
          int h = max(hv, max(ev, fv));
          En[d] = (int16_t)ev;
          Fn[d] = (int16_t)fv;
          if (h >= 0) h = extend<PK>(qs, rs, h, d, lim);
          Hn[d] = (int16_t)h;
        }
      }
    }
    if (__builtin_amdgcn_readfirstlane(end) >= M || s >= smax) {
      outgrown = false;
      break;
    }
    if (outgrown) break;
    __syncthreads();
    ++s;
  }
  if (tid == 0) {
    if (outgrown) {
      res->flags |= ALN_F_WIDENED;
    } else {
      res->score = -s * a.pen_g;
      res->q_end = M;
      res->r_end = N;
      res->cells = entries(M, N, E * a.pen_g, s * a.pen_g);
    }
  }
}

template <typename K>
static hipError_t launch_search_k(K kern, int threads, size_t lds, const SearchArgs &a,
                                  hipStream_t s) {
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(a.ntasks), dim3(threads), lds, s, a);
  return hipGetLastError();
}

#define SEARCH_LAUNCH(K, NWV, LDS)                                        \
  (a.two_bit ? launch_search_k((K<NWV, true>), 64 * NWV, (LDS), a, s) \
             : launch_search_k((K<NWV, false>), 64 * NWV, (LDS), a, s))
template <int NWV>
static hipError_t launch_search_group(const SearchArgs &a, hipStream_t s) {
  const size_t lds = (size_t)a.lds_q + a.lds_r + 2 * (size_t)a.lds_f;
  if (a.two_bit) return launch_search_k(search_group_kernel<NWV, true, false>, 64 * NWV, lds, a, s);
  return a.dcap > 0 ? launch_search_k(search_group_kernel<NWV, false, true>, 64 * NWV, lds, a, s)
                    : launch_search_k(search_group_kernel<NWV, false, false>, 64 * NWV, lds, a, s);
}
hipError_t launch_search(const SearchArgs &a, hipStream_t s) {
  if (a.ntasks <= 0) return hipSuccess;
  const size_t one = (size_t)a.lds_q + a.lds_r + a.lds_f;
  if (a.pen_x > 0) {
    if (a.pen_e <= 0 || a.pen_g <= 0 || a.ring_h < 1 || a.ring_e < 1) return hipErrorInvalidValue;
    const size_t lds = (size_t)a.lds_q + a.lds_r + (size_t)(a.ring_h + 2 * a.ring_e) * a.lds_f;
    switch (a.waves) {
    case 1: return SEARCH_LAUNCH(search_affine_kernel, 1, lds);
    case 2: return SEARCH_LAUNCH(search_affine_kernel, 2, lds);
    case 4: return SEARCH_LAUNCH(search_affine_kernel, 4, lds);
    case 8: return SEARCH_LAUNCH(search_affine_kernel, 8, lds);
    default: return hipErrorInvalidValue;
    }
  }
  if (a.one_row)
    return a.two_bit ? launch_search_k(search_edit_kernel<true>, 64, one, a, s)
                     : launch_search_k(search_edit_kernel<false>, 64, one, a, s);
  switch (a.waves) {
  case 1: return launch_search_group<1>(a, s);
  case 2: return launch_search_group<2>(a, s);
  case 4: return launch_search_group<4>(a, s);
  case 8: return launch_search_group<8>(a, s);
  default: return hipErrorInvalidValue;
  }
}
#undef SEARCH_LAUNCH

} // namespace alnk
