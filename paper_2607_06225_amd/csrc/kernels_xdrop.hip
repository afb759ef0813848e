// kernels_xdrop.hip -- X-drop seed extension on gfx950: sixteen, eight or four
// extension sides per wavefront, a persistent work queue.
//
// The rule (Sec. 2, Sec. 5.2, Sec. 7.2) evaluated antidiagonal by
// antidiagonal k = i + j in sheared coordinates d = j - i (Sec. 6.2): a
// candidate cell is removed when its H falls more than X below the best score
// of the earlier antidiagonals, and the next antidiagonal is evaluated from
// one step before the first survivor to one step after the last.
//
// Layout.  A side owns a window of 128 diagonals d = base + 2*pos + (k & 1),
// pos = 0..63: the 64 cells of one antidiagonal, XC = 16, 8 or 4 per lane on a
// group of LPS = 4, 8 or 16 lanes (lane g holds pos XC g .. XC g + XC - 1).
// (Z-drop also 256 diagonals on eight lanes.)  Per diagonal a lane keeps the
// latest H and the E / F values it passes right / down; E comes from d - 1
// and F from d + 1 of the previous antidiagonal (the other parity), H of the
// diagonal predecessor from the same slot, so one DPP per antidiagonal
// moves a value across a lane boundary.
//
// What bounds it: instruction issue when the wavefronts fill the SIMDs (0.2 to
// 0.26 VALU instructions a SIMD cycle), the chain of one step's instructions
// (about 8 cycles each for a lone wavefront) when they do not, so the step's
// instruction count either way.  Besides the 9.5 a cell, a step takes the
// side's bookkeeping, which the fields qi and rj below keep short (matrix
// edges, end cell and ring addresses are one sum each), one code read, as only
// one of the two code runs moves, and a slide of the window.  100 000 sides of
// 150..5 000 bp at X = 100: 290 instructions a step and 21.1 ms before, 240
// and 18.4 ms; 25 000 with codes 19.9 ms on four lanes a side before, 15.0 ms
// (on eight).  Z-drop, eight sides of 128 cells a wavefront: 436 instructions a step
// and 16.6 ms for 25 000 sides with the range a bit test a cell and the best key
// selected, 335 and 15.2 with the range an add's carry and the key of the masked H.
//
// Offset frame.  Every stored value of antidiagonal k is kept minus k*e (e
// the gap extension score), so a gap step adds nothing:
//   E'(k, d) = max(E'(k-1, d-1), H'(k-1, d-1) + o),  F' likewise from d+1,
//   H'(k, d) = max(H'(k-2, d) + s - 2e, E'(k, d), F'(k, d)),
// with o the gap open score.  Per cell: one add of the substitution byte
// (SDWA), a three-way max, the prune compare and select, the open add and
// two max.
//
// Pruning without range masks.  Only H of a removed cell is set to minus
// infinity.  Its E and F may keep values, but every such value is below the
// threshold of its antidiagonal, and thresholds (in the offset frame) never
// fall, so no later survivor's H, no prune decision and no survivor range
// can change.  A cell outside the candidate range inside the matrix can only
// be revived through its diagonal predecessor; its substitution score is
// replaced by -128, which keeps it below the threshold whenever
// X < 128 + 2|e| (the planner checks this).  Cells past the matrix's far
// edges (j > N or i > M) can hold values carried out of the last column or
// row; they never count as survivors, values never flow back from them, and
// with non-positive gap scores they never beat the cell they came from, so
// they never become the best cell either.
//
// Substitution scores come from one v_perm_b32 per four cells: the codes'
// XOR selects byte 0 (match) or 1..3 (mismatch) of a table, byte 4..7
// (-128) where the candidate range excludes the cell.  Codes are staged per
// side in LDS rings (query reversed) and read as one unaligned 16-byte run
// per lane and antidiagonal.
//
// Traceback codes (the form with CIGAR): per antidiagonal and side only the
// 8-cell groups (one code dword each) that hold candidate cells, packed one
// antidiagonal after the other; per antidiagonal a byte with its first and
// last group and the window base's step, per 64 antidiagonals the stream
// offset and the window base (the layout of xdl_tb_table / xdl_tb_stream).
// The cell at pos p sits in group p >> 3 at nibble 7 - (p & 7); its bits, high to low: F passed down opened from H (F-open), E passed right
// opened from H (E-open), H not from E, H not from the diagonal -- so H takes
// the diagonal, then E, then F, and a gap opens before it extends.  The codes
// of a survivor are those of the pruned recurrence: every value compared on
// the optimal path is at or above its antidiagonal's threshold, hence not a
// stale one.
//
// Best cell: keys (H' << 6 | pos) give, per antidiagonal, the highest score
// and among equals the largest d (smallest i); over antidiagonals the running
// best takes an equal score only at a smaller i (at the same i a later
// antidiagonal's j is larger).  Survivor bounds come from per-lane survivor
// masks and DPP minima / maxima.  The window slides by eight cells, or by one,
// when the candidate range reaches an edge; a wider region goes to the
// widening queue (the one-side kernel with wider windows).
#include "internal.h"

#include <type_traits>

namespace alnk {

namespace {

constexpr int XNEG = -(1 << 22);   // minus infinity in the offset frame
constexpr int XBIG = (1 << 29);    // threshold of an idle side: nothing survives
constexpr int kRingMirror = 32;    // first bytes repeated after a ring
constexpr int kSlide = 8;          // cells a window slides by where its candidates allow it
constexpr int kAhead = 20;         // codes a ring is kept ahead of the window
constexpr int kZBias = 1 << 20;    // Z-drop: bias of diagonal differences

// codes per ring: the window, its lead and a slide back fit (64 cells: 51 + 8
// + 63 < 128, 128 cells: 51 + 8 + 127 < 256)
constexpr int lanes_ring(int window) { return 2 * window; }
constexpr int lanes_lds_bytes(int lps, int window) {
  return (64 / lps) * 2 * (lanes_ring(window) + kRingMirror);
}

// Moves within a side's group of L lanes (4, 8 or 16: inside one DPP row).
// quad_perm always names a lane of the quad, so every lane reads a defined
// value and bound_ctrl changes nothing; with it and no old value the compiler
// folds the move into the instruction that uses it.
template <int CTRL> __device__ __forceinline__ int row_dpp(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
// lane l reads lane l-1 (shr) / l+1 (shl) of its group; the group's edge lane
// gets `edge`
template <int L> __device__ __forceinline__ int grp_shr1(int v, int edge, bool first) {
  if (L == 16) return __builtin_amdgcn_update_dpp(edge, v, 0x111, 0xf, 0xf, false); // row_shr:1
  const int x = L == 4 ? row_dpp<0x90>(v) : row_dpp<0x111>(v); // quad_perm 0,0,1,2
  return first ? edge : x;
}
template <int L> __device__ __forceinline__ int grp_shl1(int v, int edge, bool last) {
  if (L == 16) return __builtin_amdgcn_update_dpp(edge, v, 0x101, 0xf, 0xf, false); // row_shl:1
  const int x = L == 4 ? row_dpp<0xF9>(v) : row_dpp<0x101>(v); // quad_perm 1,2,3,3
  return last ? edge : x;
}
// every lane of the group: the group's maximum / minimum
template <int L> __device__ __forceinline__ int grp_max(int v) {
  v = max(v, row_dpp<0xB1>(v));               // quad_perm 1,0,3,2
  v = max(v, row_dpp<0x4E>(v));               // quad_perm 2,3,0,1
  if (L >= 8) v = max(v, row_dpp<0x141>(v));  // row_half_mirror
  if (L >= 16) v = max(v, row_dpp<0x140>(v)); // row_mirror
  return v;
}
template <int L> __device__ __forceinline__ uint32_t grp_umin(uint32_t v) {
  v = min(v, (uint32_t)row_dpp<0xB1>((int)v));
  v = min(v, (uint32_t)row_dpp<0x4E>((int)v));
  if (L >= 8) v = min(v, (uint32_t)row_dpp<0x141>((int)v));
  if (L >= 16) v = min(v, (uint32_t)row_dpp<0x140>((int)v));
  return v;
}

// 4 NW ring bytes from `addr`, any alignment (the mirror covers the wrap): one
// unaligned LDS read of 8 or 16 bytes; for 4 bytes two aligned dwords and a
// byte align, which take less time (4.4 against 4.8 ms for 400 sides alone)
template <int NW>
__device__ __forceinline__ void ring_read(const uint8_t *ring, int addr, uint32_t (&w)[NW]) {
  if constexpr (NW == 1) {
    const uint32_t *d = reinterpret_cast<const uint32_t *>(ring + (addr & ~3));
    w[0] = __builtin_amdgcn_alignbyte(d[1], d[0], (uint32_t)addr & 3u);
  } else {
    __builtin_memcpy(w, ring + addr, 4 * NW);
  }
}

// v = 2 v + bit, the bit taken from a compare's lane mask as a carry
__device__ __forceinline__ void shift_in(uint32_t &v, bool bit) {
  const unsigned long long km = __builtin_amdgcn_ballot_w64(bit);
  unsigned long long cc;
  asm("v_addc_co_u32_e64 %0, %1, %2, %2, %3" : "=v"(v), "=s"(cc) : "v"(v), "s"(km));
  (void)cc;
}

// the lane mask of v's top bits, and v = 2 v: one add and its carry
__device__ __forceinline__ unsigned long long shift_out(uint32_t &v) {
  unsigned long long m;
  asm("v_add_co_u32_e64 %0, %1, %2, %2" : "=v"(v), "=s"(m) : "v"(v));
  return m;
}

// byte b of the result = byte 3 - b of x
__device__ __forceinline__ uint32_t byte_reverse(uint32_t x) {
  return __builtin_amdgcn_perm(0u, x, 0x00010203u);
}

} // namespace

// LPS lanes a side, XC cells a lane: a window of W = LPS * XC cells.
// ZD: Z-drop (Sec. 9.3) instead of X-drop: a candidate is kept when its H
// plus its distance |d - d_best| from the best cell's diagonal reaches the
// threshold.  The thresholds then differ between diagonals, so the pruning
// above is made explicit: H, E and F of a removed cell or of a cell outside
// the candidate range are minus infinity, and only kept cells enter the
// antidiagonal's best.
template <int LPS, int XC, bool TB, bool ZD>
__device__ __forceinline__ void lanes_body(const XdlArgs &a, uint8_t *smem) {
  constexpr int W = LPS * XC;          // cells of a side's window
  constexpr int PB = W == 64 ? 6 : 7;  // bits of a position
  constexpr int NW = XC / 4;           // code dwords a lane reads
  constexpr int kRing = lanes_ring(W);
  constexpr int kRingStride = kRing + kRingMirror;
  constexpr int kStageB = 32 / LPS;    // codes a lane stages at a time
  // the candidate range of the widest antidiagonal kept here: the window for
  // X-drop, 126 cells (a range of 250 diagonals, as the one-side kernel's
  // first window) for the wide window
  constexpr int kWidest = W == 64 ? 64 : 126;
  static_assert(W == 64 || W == 128, "positions are 6 or 7 bits");
  static_assert(!TB || W == 64, "the code layout is that of 64-cell windows");
  const int lane = threadIdx.x & 63;
  const int gl = lane & (LPS - 1); // lane within the side's group
  const int side = lane / LPS;     // side slot of this wavefront
  const bool qfirst = gl == 0, qlast = gl == LPS - 1;
  uint8_t *qring = smem + side * 2 * kRingStride;
  uint8_t *rring = qring + kRingStride;

  const int X = a.xdrop, go = a.gap_open, ge = a.gap_extend;
  // substitution table in the offset frame: byte 0 match, 1..3 mismatch,
  // 4..7 the out-of-range penalty
  const uint32_t m8 = (uint32_t)(a.match - 2 * ge) & 0xffu;
  const uint32_t x8 = (uint32_t)(a.mismatch - 2 * ge) & 0xffu;
  const uint32_t tab_lo = m8 | (x8 << 8) | (x8 << 16) | (x8 << 24);
  const uint32_t tab_hi = 0x80808080u;

  int H0[XC], H1[XC], E0[XC], F0[XC], E1[XC], F1[XC];
#pragma unroll
  for (int m = 0; m < XC; ++m) H0[m] = H1[m] = E0[m] = F0[m] = E1[m] = F1[m] = XNEG;

  // Side state, equal across the group.  qi, rj: row and column of the cell
  // at pos 0 (pos p is cell (qi - p, rj + p) of antidiagonal k = qi + rj, on
  // diagonal base + 2p + (k & 1), base = rj - qi - (k & 1)); an odd
  // antidiagonal's rj, an even one's qi is one more than the antidiagonal's
  // before.
  bool active = false, exhausted = false;
  int task = 0, pair = 0, M = 0, N = 0, qi = 0, rj = 0;
  int plo = 1, phi = 0, qtop = 0, rtop = 0;
  int bk = XBIG;              // best score so far, in the antidiagonal's frame
  int best_i = 0, best_j = 0; // its cell
  int cells = 0;              // at most 126 * (M + N) < 2^31
  // codes of this lane's cells, kept from one antidiagonal to the next
  uint32_t qw[NW], rw[NW];
  bool reload = true; // wave-uniform: some side's window moved, or is new
  const uint8_t *Q = nullptr, *R = nullptr;
  // traceback: one byte per antidiagonal, a table entry per 64, the codes
  uint8_t *tb_meta = nullptr; // the side's region
  int tcur = 0;               // byte offset in the region of the next code dword
  uint32_t sbits = 0;         // the window base's step (bits 6-7 of the byte)
  uint32_t mlo = 0, mhi = 0;  // lane gl: bytes of antidiagonals 32n + 8gl .. + 7, newest on top

  // 32 codes per call into a ring (the query reversed), padding (4) past
  // the sequence; lane gl stages kStageB of them
  auto stage = [&](const uint8_t *src, int len, uint8_t *ring, int top, bool rev) {
    const int c0 = top + kStageB * gl;
    uint32_t w[2] = {0, 0};
#pragma unroll
    for (int b = 0; b < kStageB; ++b) {
      const int c = c0 + b;
      const uint32_t raw = src[min(c, len - 1)]; // clamped: issued unconditionally
      const uint32_t v = (c < len) ? min(raw, 4u) : 4u;
      const int at = rev ? kStageB - 1 - b : b; // byte of the stored run
      w[at >> 2] |= v << (8 * (at & 3));
    }
    // reversed: code c lives at (kRing - 1 - c) mod kRing
    const int at = rev ? (kRing - kStageB - (c0 & (kRing - 1))) & (kRing - 1) : c0 & (kRing - 1);
    auto put = [&](uint8_t *dst) {
      if constexpr (kStageB == 8) *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
      else if constexpr (kStageB == 4) *reinterpret_cast<uint32_t *>(dst) = w[0];
      else *reinterpret_cast<uint16_t *>(dst) = (uint16_t)w[0];
    };
    put(ring + at);
    if (at < kRingMirror) put(ring + kRing + at);
  };

  for (;;) {
    // ---- idle sides take the next task (the list is longest first)
    bool need = !active && !exhausted;
    bool fresh = false;
    while (__ballot(need)) {
      if (need) {
        int t = 0;
        if (qfirst) t = atomicAdd(a.queue, 1);
        t = LPS == 4 ? row_dpp<0x00>(t) : __shfl(t, lane & ~(LPS - 1), 64); // the first lane's
        if (t >= a.ntasks) {
          exhausted = true;
        } else {
          task = t;
          pair = a.tasks[t].pair;
          M = a.b.q_len[pair];
          N = a.b.r_len[pair];
          if (M == 0 || N == 0) {
            if (qfirst) {
              aln_result *res = a.res + pair;
              res->score = 0;
              res->q_end = 0;
              res->r_end = 0;
              res->cells = 0;
            }
          } else {
            Q = a.b.q + a.b.q_off[pair];
            R = a.b.r + a.b.r_off[pair];
            if (TB) {
              const int nb = (M + N + 1 + 63) / 64;
              uint8_t *tbp = a.tb + a.tasks[t].tb_off;
              tb_meta = tbp;
              tcur = (int)xdl_tb_stream(nb);
              sbits = 0;
              mlo = 0;
              mhi = 1u << 24; // antidiagonal 0: no groups (first 1, last 0)
              if (qfirst) *reinterpret_cast<int2 *>(tbp + xdl_tb_table(nb)) = make_int2(0, -W);
            }
            fresh = true; // arrays reset below, outside this loop
            qi = W / 2; // k = 1, base -W
            rj = 1 - W / 2;
            bk = -ge; // score 0 at (0,0)
            best_i = best_j = 0;
            plo = W / 2 - 1; // candidates of k = 1: d = -1, 1
            phi = W / 2;
            cells = 0;
            qtop = 0;
            rtop = 0;
            // rings start as padding
            for (int e = gl * 4; e < 2 * kRingStride; e += 4 * LPS)
              *reinterpret_cast<uint32_t *>(qring + e) = 0x04040404u;
            active = true;
          }
        }
      }
      need = !active && !exhausted;
    }
    if (!__ballot(active)) break;
    // new sides: every slot minus infinity but the cell (0,0) with H = 0 at
    // d = 0 (pos W / 2, parity 0), whose E and F outputs are the gap open in the
    // frame of k = 1
    if (__ballot(fresh)) {
      reload = true;
      if (fresh) {
#pragma unroll
        for (int m = 0; m < XC; ++m) H0[m] = H1[m] = E0[m] = F0[m] = E1[m] = F1[m] = XNEG;
        if (gl == LPS / 2) {
          H0[0] = 0;
          E0[0] = go;
          F0[0] = go;
        }
      }
    }

    // one antidiagonal of parity P (the antidiagonal's, for every active side)
    auto step = [&](auto ptag) {
      constexpr int P = decltype(ptag)::value;
      // ---- keep the rings ahead of the window: the codes read before the
      // next check lie at most 10 past the top (a slide of 8 and one
      // antidiagonal each way), and a ring filled to 51 past it still holds the
      // window's last code after a slide back by 8 (51 + 8 + 63 < 128; further
      // slides back take at least as many antidiagonals as they move)
      for (; P == 1;) {
        const int topq = qi - 1;     // query code of pos 0
        const int topr = rj + W - 2; // reference code of the last pos
        const bool sq = active && qtop < topq + kAhead;
        const bool sr = active && rtop < topr + kAhead;
        if (!__ballot(sq || sr)) break;
        if (sq) {
          stage(Q, M, qring, qtop, true);
          qtop += 32;
        }
        if (sr) {
          stage(R, N, rring, rtop, false);
          rtop += 32;
        }
      }
      // ---- this lane's codes: query i - 1 (descending) and reference j - 1.
      // One of the two runs moves by one code an antidiagonal, so it alone is
      // read, one antidiagonal ahead (below); both after a slide.
      auto read_q = [&](uint32_t(&w)[NW], int ahead) {
        ring_read<NW>(qring, (kRing - (qi + ahead) + XC * gl) & (kRing - 1), w);
      };
      auto read_r = [&](uint32_t(&w)[NW], int ahead) {
        ring_read<NW>(rring, (rj + ahead - 1 + XC * gl) & (kRing - 1), w);
      };
      if (reload) {
        read_q(qw, 0);
        read_r(rw, 0);
        reload = false;
      }
      // ---- substitution bytes; cells outside [plo, phi] get the penalty
      uint32_t sc[NW], inr_rev; // inr_rev: bit XC - 1 - m set for cells m in range
      {
        const int lo = min(max(plo - XC * gl, 0), XC);
        const int hi = min(max(phi - XC * gl + 1, 0), XC);
        // hi >= lo always (an idle side has plo = phi + 1)
        const uint32_t in = (1u << (hi - lo)) - 1u;
        inr_rev = in << (XC - hi);
        const uint32_t out = ~(in << lo);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          const uint32_t nib = (out >> (4 * w)) & 15u;
          const uint32_t spread = __umul24(nib, 0x00810204u) & 0x04040404u; // bit 2 of each byte
          sc[w] = __builtin_amdgcn_perm(tab_hi, tab_lo, (qw[w] ^ rw[w]) | spread);
        }
      }
      uint32_t nw[NW]; // the run that moves next, read now
      if (P == 1) read_q(nw, 1);
      else read_r(nw, 1);
      const int T = bk - X;
      // ---- the cells
      int kmax = INT32_MIN;
      uint32_t sb = 0, code0 = 0, code1 = 0;
      // Z-drop: this lane's first cell's diagonal minus the best cell's,
      // biased so that the distance is one unsigned difference per cell
      uint32_t zlane = 0, zin = inr_rev << (32 - XC); // cells in range, from the top
      if (ZD) {
        zlane = (uint32_t)(rj - qi + 2 * XC * gl - (best_j - best_i) + kZBias);
      }
      const int xin = P == 0 ? grp_shr1<LPS>(E1[XC - 1], XNEG, qfirst)
                             : grp_shl1<LPS>(F0[0], XNEG, qlast);
#pragma unroll
      for (int m = 0; m < XC; ++m) {
        const int ein = P == 0 ? (m == 0 ? xin : E1[m - 1]) : E0[m];
        const int fin = P == 0 ? F1[m] : (m == XC - 1 ? xin : F0[m + 1]);
        const int hp = P == 0 ? H0[m] : H1[m];
        const int s = (int)(int8_t)(sc[m >> 2] >> (8 * (m & 3)));
        const int h = max(max(hp + s, ein), fin);
        bool keep = h >= T;
        if (ZD) {
          // h + |d - d_best|, d = (first cell's diagonal) + 2m
          const uint32_t zc = (uint32_t)(kZBias - 2 * m);
          const int hz = (int)((max(zlane, zc) - min(zlane, zc)) + (uint32_t)h);
          keep = __builtin_amdgcn_inverse_ballot_w64(__builtin_amdgcn_ballot_w64(hz >= T) & shift_out(zin));
        }
        const int hm = keep ? h : XNEG;
        // X-drop: E and F may take h of a removed cell, below the threshold
        // either way
        const int t = h + go;
        const int en = (ZD && !keep) ? XNEG : max(ein, t);
        const int fn = (ZD && !keep) ? XNEG : max(fin, t);
        if (P == 0) {
          H0[m] = hm;
          E0[m] = en;
          F0[m] = fn;
        } else {
          H1[m] = hm;
          E1[m] = en;
          F1[m] = fn;
        }
        // a removed cell never beats a kept one (X-drop: nor does its h)
        kmax = max(kmax, ((ZD ? hm : h) << PB) | m);
        // shift the survivor bit in: sb = 2 sb + keep (cell m ends at bit XC - 1 - m)
        shift_in(sb, keep);
        if (TB) { // the cell's code, high bit first
          uint32_t &c = m < 8 ? code0 : code1;
          shift_in(c, t >= fin);
          shift_in(c, t >= ein);
          shift_in(c, ein < h);
          shift_in(c, hp + s < h);
        }
      }
      if (TB && active) {
        // only the 8-cell groups g0 .. g1 that hold candidates are stored
        // (a walk reads survivors only), after the antidiagonal before's
        const int g0 = plo >> 3, span = (phi >> 3) - g0;
        // stream slot of this lane's first group (4 cells a lane: the even
        // lane holds its group's upper half)
        const int e0 = XC * gl / 8 - g0;
        uint8_t *dst = tb_meta + (tcur + 4 * e0);
        if ((unsigned)e0 <= (unsigned)span) {
          if constexpr (XC == 4) *reinterpret_cast<uint16_t *>(dst + ((gl & 1) ? 0 : 2)) = (uint16_t)code0;
          else *reinterpret_cast<uint32_t *>(dst) = code0;
        }
        if (XC == 16 && (unsigned)(e0 + 1) <= (unsigned)span)
          *reinterpret_cast<uint32_t *>(dst + 4) = code1;
        tcur += 4 * (span + 1);
        // the antidiagonal's byte: g0 (bits 0-2), g1 (3-5) and the window
        // base's step from the antidiagonal before, (base - bprev) / 2 in
        // two's complement (bits 6-7).  Lane gl collects those of its 8 of
        // every 32 antidiagonals, and the side's first four lanes store the 32
        // bytes at once (one whole memory sector: smaller stores cost as
        // much each)
        const int k = qi + rj;
        const uint32_t mbyte = ((uint32_t)plo >> 3) | ((uint32_t)phi & 0x38u) | sbits;
        sbits = 0;
        if (((k >> 3) & 3) == gl) {
          mlo = __builtin_amdgcn_alignbit(mhi, mlo, 8);
          mhi = __builtin_amdgcn_alignbit(mbyte, mhi, 8);
        }
        if ((k & 31) == 31) {
          if (gl < 4) *reinterpret_cast<uint2 *>(tb_meta + (k - 31) + 8 * gl) = make_uint2(mlo, mhi);
          if ((k & 63) == 63) {
            // the next block starts on a 16-byte boundary; its entry holds
            // the base of its antidiagonal before (the table has room for
            // one entry past the last block)
            tcur = (tcur + 15) & ~15;
            const int nb = (M + N + 64) >> 6;
            if (qfirst)
              reinterpret_cast<int2 *>(tb_meta + xdl_tb_table(nb))[(k + 1) >> 6] =
                  make_int2((tcur - (int)xdl_tb_stream(nb)) >> 2, rj - qi - P);
          }
        }
      }
      sb &= inr_rev;
      // ---- the antidiagonal's outcome per side
      kmax = grp_max<LPS>(kmax | (XC * gl));
      // first and last survivor: bit counts of an empty lane read 2^32 - 1 and
      // saturate to a position that never wins (no survivor at all: f > l)
      const uint32_t sb32 = sb << (32 - XC);
      const uint32_t c1 = sb ? (uint32_t)__builtin_clz(sb32) : ~0u;
      const uint32_t c0 = sb ? (uint32_t)__builtin_ctz(sb) : ~0u;
      const uint32_t fl = __builtin_elementwise_add_sat((uint32_t)(XC * gl), c1);
      const uint32_t ll = __builtin_elementwise_sub_sat((uint32_t)(XC * gl + XC - 1), c0);
      const int f = (int)grp_umin<LPS>(fl), l = grp_max<LPS>((int)ll);
      const bool surv = active && (uint32_t)f <= (uint32_t)l;
      {
        // (without survivors every score is below T <= bk)
        const int hs = kmax >> PB, ps = kmax & (W - 1);
        const int bi = qi - ps;
        // equal score: the smaller i (of one i, the earlier antidiagonal's j
        // is the smaller)
        const bool up = hs > bk || (hs == bk && bi < best_i);
        best_i = up ? bi : best_i;
        best_j = up ? rj + ps : best_j;
        bk = max(bk, hs);
      }
      // ---- next antidiagonal: candidates in the other parity's positions,
      // clipped to the matrix (0 <= i <= M, 0 <= j <= N)
      const int qn = P == 1 ? qi + 1 : qi, rn = P == 1 ? rj : rj + 1;
      const int nlo = max(max(P == 0 ? f - 1 : f, -rn), qn - M);
      const int nhi = min(min(P == 0 ? l : l + 1, qn), N - rn);
      const bool cont = surv && nlo <= nhi;
      const bool wide = cont && nhi - nlo >= kWidest;
      if (active && (!cont || wide)) {
        // the extension ends here (or leaves for a wider window)
        const int k = qi + rj;
        if (TB && gl < 4 && (k & 31) != 31 && 8 * gl <= (k & 31)) { // the bytes of the last, partial 32
          const int sh = 8 * gl + 7 > (k & 31) ? 8 * (7 - (k & 7)) : 0; // a partial 8
          const unsigned long long m8 = ((unsigned long long)mhi << 32 | mlo) >> sh;
          *reinterpret_cast<uint2 *>(tb_meta + (k & ~31) + 8 * gl) =
              make_uint2((uint32_t)m8, (uint32_t)(m8 >> 32));
        }
        if (qfirst) {
          aln_result *res = a.res + pair;
          if (wide) {
            // score only: the wider one-side kernel; with traceback: the
            // one-side pass that writes codes in its own layout (the walk of
            // this layout skips the pair, marked in its task)
            res->flags |= ALN_F_WIDENED;
            const int slot = atomicAdd(a.widen_count, 1);
            const PairTask *src = a.tasks + task;
            PairTask *dst = a.widen + slot;
            dst->pair = src->pair;
            dst->rows = a.widen_rows;
            dst->tb_off = src->tb_off;
            dst->cigar_off = src->cigar_off;
            dst->cigar_cap = src->cigar_cap;
            dst->aux = 0;
            if (TB) const_cast<PairTask *>(a.tasks)[task].aux = 1;
          } else {
            res->score = bk + k * ge;
            res->q_end = best_i;
            res->r_end = best_j;
            res->cells = cells;
          }
        }
        active = false;
        bk = XBIG;
      }
      // (an idle side keeps an empty range and a threshold nothing reaches)
      plo = active ? nlo : 1;
      phi = active ? nhi : 0;
      // interior cells (i, j >= 1) of the next antidiagonal
      cells += max(min(phi, qn - 1) - max(plo, 1 - rn) + 1, 0);
      qi = qn;
      rj = rn;
      bk -= ge;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        if (P == 1) qw[w] = nw[w];
        else rw[w] = nw[w];
      }
      // ---- keep the candidates inside the window.  The live arrays are both
      // H and the E / F just written.  A side whose candidates leave it slides
      // by eight cells where they still fit then, else by one: with sixteen
      // sides a wavefront, slides of one cell came on nearly every
      // antidiagonal and were 40% of the kernel's instructions (344 a step,
      // 205 without them; 400 000 sides of 150..5 000 bp, X = 100).
      const bool sup = active && plo < 0, sdn = active && phi >= W;
      const bool sup8 = sup && phi + kSlide < W - (TB ? kSlide : 0); // TB: see mbyte
      const bool sdn8 = sdn && plo >= kSlide;
      // The shifts are selects in place under a wave-uniform branch: a
      // branch on the side's own flag made the compiler copy every array at
      // its join on every antidiagonal (about 100 moves per lane).
      auto slide_up = [&](int(&A)[XC], bool on, auto by_tag) { // every pos moves up
        constexpr int S = decltype(by_tag)::value, SL = S / XC, SC = S % XC; // lanes, cells
        int v[XC]; // moved by whole lanes
#pragma unroll
        for (int m = 0; m < XC; ++m) {
          v[m] = A[m];
#pragma unroll
          for (int t = 0; t < SL; ++t) v[m] = grp_shr1<LPS>(v[m], XNEG, qfirst);
        }
        int c[SC + 1];
#pragma unroll
        for (int m = 0; m < SC; ++m) c[m] = grp_shr1<LPS>(v[XC - SC + m], XNEG, qfirst);
#pragma unroll
        for (int m = XC - 1; m >= SC; --m) A[m] = on ? v[m - SC] : A[m];
#pragma unroll
        for (int m = 0; m < SC; ++m) A[m] = on ? c[m] : A[m];
      };
      auto slide_down = [&](int(&A)[XC], bool on, auto by_tag) { // every pos moves down
        constexpr int S = decltype(by_tag)::value, SL = S / XC, SC = S % XC;
        int v[XC];
#pragma unroll
        for (int m = 0; m < XC; ++m) {
          v[m] = A[m];
#pragma unroll
          for (int t = 0; t < SL; ++t) v[m] = grp_shl1<LPS>(v[m], XNEG, qlast);
        }
        int c[SC + 1];
#pragma unroll
        for (int m = 0; m < SC; ++m) c[m] = grp_shl1<LPS>(v[m], XNEG, qlast);
#pragma unroll
        for (int m = 0; m < XC - SC; ++m) A[m] = on ? v[m + SC] : A[m];
#pragma unroll
        for (int m = 0; m < SC; ++m) A[XC - SC + m] = on ? c[m] : A[XC - SC + m];
      };
      using One = std::integral_constant<int, 1>;
      using Many = std::integral_constant<int, kSlide>;
      auto up_all = [&](bool on, auto by_tag) { // base falls
        constexpr int S = decltype(by_tag)::value;
        slide_up(H0, on, by_tag);
        slide_up(H1, on, by_tag);
        slide_up(P == 0 ? E0 : E1, on, by_tag);
        slide_up(P == 0 ? F0 : F1, on, by_tag);
        qi += on ? S : 0;
        rj -= on ? S : 0;
        plo += on ? S : 0;
        phi += on ? S : 0;
        if (TB) sbits = on ? (S == 1 ? 0xc0u : 0x80u) : sbits;
      };
      auto down_all = [&](bool on, auto by_tag) { // base rises
        constexpr int S = decltype(by_tag)::value;
        slide_down(H0, on, by_tag);
        slide_down(H1, on, by_tag);
        slide_down(P == 0 ? E0 : E1, on, by_tag);
        slide_down(P == 0 ? F0 : F1, on, by_tag);
        qi -= on ? S : 0;
        rj += on ? S : 0;
        plo -= on ? S : 0;
        phi -= on ? S : 0;
        if (TB) sbits = on ? (S == 1 ? 0x40u : 0x80u) : sbits;
      };
      if (__ballot(sup || sdn)) {
        reload = true;
        if (__ballot(sup8)) up_all(sup8, Many{});
        if (__ballot(sdn8)) down_all(sdn8, Many{});
        if (__ballot(sup && !sup8)) up_all(sup && !sup8, One{});
        if (__ballot(sdn && !sdn8)) down_all(sdn && !sdn8, One{});
      }
    };
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 0>{});
  }
  // the last wavefront out resets the queue for the next launch
  if (lane == 0 && atomicAdd(a.queue + 1, 1) == (int)gridDim.x - 1) {
    a.queue[0] = 0;
    a.queue[1] = 0;
  }
}

// Sixteen cells a lane: four wavefronts per SIMD for the X-drop score form
// (128 VGPRs, no spill in the step), three with codes or Z-drop (they need more
// registers).  Fewer cells a lane take fewer registers (xdrop_lanes_waves).
template <int LPS, int XC, bool TB, bool ZD>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(xdrop_lanes_waves(TB, ZD, LPS) / 4))) void
xdrop_lanes_kernel(XdlArgs a) {
  extern __shared__ __align__(16) uint8_t smem[];
  lanes_body<LPS, XC, TB, ZD>(a, smem);
}

template <int LPS, int XC, bool TB, bool ZD>
static hipError_t launch_lanes(const XdlArgs &a, int waves, hipStream_t s) {
  hipLaunchKernelGGL((xdrop_lanes_kernel<LPS, XC, TB, ZD>), dim3(waves), dim3(64),
                     (size_t)lanes_lds_bytes(LPS, LPS * XC), s, a);
  return hipGetLastError();
}

// Forms by lanes a side: 4, 8 or 16 of a 64-cell window (X-drop, with codes or
// without; Z-drop without codes: 4), or 8 of a 128-cell window (Z-drop).
hipError_t launch_xdrop_lanes(bool tb, const XdlArgs &a, int waves, hipStream_t s) {
  if (a.ntasks <= 0) return hipSuccess;
  if (a.zdrop) { // Z-drop codes: the one-side pass
    if (tb) return hipErrorInvalidValue;
    if (a.window == 128 && a.lps == 8) return launch_lanes<8, 16, false, true>(a, waves, s);
    if (a.window == 64 && a.lps == 4) return launch_lanes<4, 16, false, true>(a, waves, s);
    return hipErrorInvalidValue;
  }
  if (a.window != 64) return hipErrorInvalidValue;
  switch (a.lps) {
  case 4: return tb ? launch_lanes<4, 16, true, false>(a, waves, s) : launch_lanes<4, 16, false, false>(a, waves, s);
  case 8: return tb ? launch_lanes<8, 8, true, false>(a, waves, s) : launch_lanes<8, 8, false, false>(a, waves, s);
  case 16: return tb ? launch_lanes<16, 4, true, false>(a, waves, s) : launch_lanes<16, 4, false, false>(a, waves, s);
  default: return hipErrorInvalidValue;
  }
}

} // namespace alnk
