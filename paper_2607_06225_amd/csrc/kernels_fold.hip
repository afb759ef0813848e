// kernels_fold.hip -- Nussinov RNA folding on gfx950, unpruned or with X-drop
// pruning transferred from alignment.
//
// Recurrence (the RNA-folding row of the example-recurrence table, Sec. 3),
// for 0 <= i < j < n:
//   F(i,j) = max( F(i+1,j), F(i,j-1), F(i+1,j-1) + in1(i,j),
//                 max over i <= k < j of F(i,k) + F(k+1,j) ),
// F(i,i) = 0, the empty interval F(i+1,i) = 0.  The bifurcation terms at
// k = i and k = j-1 are F(i+1,j) and F(i,j-1) (F(i,i) = F(j,j) = 0), so the
// reduction over k covers the first two terms as well.
//
// Every term reads a shorter interval, so the cells of one span t = j - i are
// independent: one workgroup per sequence walks the spans t = 1 .. n-1 (the
// triangle's wavefronts; with rows flipped they are its antidiagonals, which
// the pruning rule of Sec. 9.5 counts) with a barrier between them.
//
// Storage: the whole triangle lives in LDS, folded into ceil(n/2) rows of a
// compile-time stride SC >= n + 1: row v holds span v (positions 0 .. n-1-v)
// followed by span n-1-v (positions 0 .. v), so F(p, p+t) sits at
//   t <  ceil(n/2):  t*SC + p
//   t >= ceil(n/2):  (n-1-t)*SC + t + 1 + p.
// For cell (i, i+t) the term of split k = i+u reads F(i, i+u) (span u,
// position i) and F(i+u+1, i+t) (span t-1-u, position i+u+1).  As u steps by
// one, each of the two addresses moves by SC (its span in the upper half of
// the rows, resp. the lower) or by 1 - SC: between the two break points u =
// ceil(n/2) and u = t - ceil(n/2) both steps are compile-time constants, so
// a block of eight splits reads with immediate offsets from two address
// registers and costs an add and a max per term.  Lanes take consecutive
// cells i, so the reads of a wave are consecutive bytes.  Elements are int16
// (minus infinity = -32768) or, when every score fits, uint8 (at most 253;
// 255 is minus infinity), which halves LDS so that 500-nt sequences fit a CU.
//
// Work split per wavefront: each wave takes 64 consecutive cells; when there
// are fewer such chunks than waves, the u-range of each chunk is split among
// waves and their partial maxima meet in LDS (one more barrier).
//
// X-drop (Sec. 7.2 rule, Sec. 9.5 transfer): candidates of span t are the
// positions from one before the first survivor of span t-1 to its last
// survivor, inside the triangle; past the warm-up (t > warmup) a cell more
// than X below the best score of the earlier spans is removed (reads as minus
// infinity).  A cell with no live term reads minus infinity too.  The result
// is the best surviving cell: highest F, then the largest span, then the
// smallest i.
//
// Unpruned sequences with byte elements take a form of their own, by tiles
// (fold_tile_kernel).
#include <algorithm>

#include "internal.h"

namespace alnk {

namespace {


// element traits: minus infinity and the per-term / final encodings
template <typename T, bool XD> struct FoldElt;
template <bool XD> struct FoldElt<int16_t, XD> {
  static constexpr int kDead = -32768;
  // term of two stored values; minus infinity stays negative
  __device__ static int term(int l, int r) { return l + r; }
  // a live result v >= 0
  __device__ static bool live(int v) { return v >= 0; }
  __device__ static int value(int v) { return v; }
  __device__ static int inner(int in, int s) { return in + s; } // in: stored F(i+1,j-1)
  static constexpr int kAccInit = -65536;
};
template <> struct FoldElt<uint8_t, true> {
  // live values 0..253, 255 = minus infinity.  A term l + r + 1 is at most
  // 254 when both are live (it is a lower bound of F(i,j) + 1) and at least
  // 256 when one is 255; read as a signed 9-bit field it is F + 1 > 0 or
  // negative.
  static constexpr int kDead = 255;
  __device__ static int term(int l, int r) {
    return __builtin_amdgcn_sbfe(l + r + 1, 0, 9);
  }
  __device__ static bool live(int v) { return v >= 1; }
  __device__ static int value(int v) { return v - 1; }
  __device__ static int inner(int in, int s) { return __builtin_amdgcn_sbfe(in + s + 1, 0, 9); }
  static constexpr int kAccInit = -1;
};

// Maximum / minimum over the wave by DPP (prefix within each 16-lane row,
// then across rows); lane 63 ends with the result.  Lanes without a source
// read the identity.
__device__ __forceinline__ int fold_wave_max(int v) {
  constexpr int id = INT32_MIN;
  v = max(v, __builtin_amdgcn_update_dpp(id, v, 0x111, 0xf, 0xf, false)); // row_shr:1
  v = max(v, __builtin_amdgcn_update_dpp(id, v, 0x112, 0xf, 0xf, false)); // row_shr:2
  v = max(v, __builtin_amdgcn_update_dpp(id, v, 0x114, 0xf, 0xf, false)); // row_shr:4
  v = max(v, __builtin_amdgcn_update_dpp(id, v, 0x118, 0xf, 0xf, false)); // row_shr:8
  v = max(v, __builtin_amdgcn_update_dpp(id, v, 0x142, 0xa, 0xf, false)); // row_bcast:15
  v = max(v, __builtin_amdgcn_update_dpp(id, v, 0x143, 0xc, 0xf, false)); // row_bcast:31
  return v;
}
__device__ __forceinline__ int fold_wave_min(int v) {
  constexpr int id = INT32_MAX;
  v = min(v, __builtin_amdgcn_update_dpp(id, v, 0x111, 0xf, 0xf, false));
  v = min(v, __builtin_amdgcn_update_dpp(id, v, 0x112, 0xf, 0xf, false));
  v = min(v, __builtin_amdgcn_update_dpp(id, v, 0x114, 0xf, 0xf, false));
  v = min(v, __builtin_amdgcn_update_dpp(id, v, 0x118, 0xf, 0xf, false));
  v = min(v, __builtin_amdgcn_update_dpp(id, v, 0x142, 0xa, 0xf, false));
  v = min(v, __builtin_amdgcn_update_dpp(id, v, 0x143, 0xc, 0xf, false));
  return v;
}

} // namespace

// Element index of F(p, p+u) in the folded triangle (H = ceil(n/2)).
template <int SC>
__device__ __forceinline__ int fold_at(int u, int p, int n, int H) {
  return u < H ? u * SC + p : (n - 1 - u) * SC + u + 1 + p;
}

// cnt splits with compile-time address steps D1 / D2, eight per block from
// the block's lowest address (immediate offsets), into two accumulators.
template <typename T, bool XD, int D1, int D2>
__device__ __forceinline__ void fold_run(const T *G, int &a1, int &a2, int cnt, int &acc0,
                                         int &acc1) {
  using E = FoldElt<T, XD>;
  constexpr int U = 8;
  for (; cnt >= U; cnt -= U) {
    // the block's lowest addresses; the empty asm keeps the compiler from
    // folding them back into one add per read (DS offsets are unsigned)
    int b1 = D1 > 0 ? a1 : a1 + (U - 1) * D1;
    int b2 = D2 > 0 ? a2 : a2 + (U - 1) * D2;
    asm volatile("" : "+v"(b1), "+v"(b2));
    const T *p1 = G + b1;
    const T *p2 = G + b2;
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int o1 = D1 > 0 ? k * D1 : (U - 1 - k) * -D1;
      const int o2 = D2 > 0 ? k * D2 : (U - 1 - k) * -D2;
      const int tv = E::term((int)p1[o1], (int)p2[o2]);
      if (k & 1) acc1 = max(acc1, tv);
      else acc0 = max(acc0, tv);
    }
    a1 += U * D1;
    a2 += U * D2;
  }
  for (; cnt > 0; --cnt) {
    acc0 = max(acc0, E::term((int)G[a1], (int)G[a2]));
    a1 += D1;
    a2 += D2;
  }
}

// Maximum over splits u in [u0, u1) of the bifurcation terms of cell (i, i+t).
template <typename T, bool XD, int SC>
__device__ __forceinline__ int fold_partial(const T *G, int n, int H, int t, int i, int u0,
                                            int u1) {
  using E = FoldElt<T, XD>;
  int acc0 = E::kAccInit, acc1 = E::kAccInit;
  int u = u0;
  int a1 = fold_at<SC>(u, i, n, H), a2 = fold_at<SC>(t - 1 - u, i + u + 1, n, H);
  while (u < u1) {
    // the segment up to the next break point: span u leaves the upper rows
    // at u = H, span t-1-u enters them at u = t - H
    int e = u1;
    if (u < H) e = min(e, H);
    if (u < t - H) e = min(e, t - H);
    const int cnt = e - u;
    const bool top1 = u < H, top2 = t - 1 - u < H;
    if (top1 && top2) fold_run<T, XD, SC, 1 - SC>(G, a1, a2, cnt, acc0, acc1);
    else if (top1) fold_run<T, XD, SC, SC>(G, a1, a2, cnt, acc0, acc1);
    else if (top2) fold_run<T, XD, 1 - SC, 1 - SC>(G, a1, a2, cnt, acc0, acc1);
    else fold_run<T, XD, 1 - SC, SC>(G, a1, a2, cnt, acc0, acc1);
    u = e;
    // crossing a break point moves an address by other than its step
    if (u < u1) {
      a1 = fold_at<SC>(u, i, n, H);
      a2 = fold_at<SC>(t - 1 - u, i + u + 1, n, H);
    }
  }
  return max(acc0, acc1);
}

template <typename T, bool XD, int B, int SC>
__global__ __launch_bounds__(B) void fold_kernel(FoldArgs a) {
  using E = FoldElt<T, XD>;
  constexpr int W = B / 64;
  extern __shared__ __align__(16) uint8_t smem[];
  const FoldTask tk = a.tasks[blockIdx.x];
  const int n = tk.n;
  const int sq = tk.seq;
  aln_fold_result *res = a.res + sq;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;

  // LDS: G (folded triangle) | codes | partial maxima (one int per cell of
  // a span) | control
  const int H = (n + 1) >> 1;
  const int gbytes = (int)(((size_t)((a.max_n + 1) >> 1) * SC * sizeof(T) + 15) & ~(size_t)15);
  T *G = reinterpret_cast<T *>(smem);
  uint8_t *xs = smem + gbytes;
  int *red = reinterpret_cast<int *>(smem + gbytes + ((n + 15) & ~15));
  int *ctl = red + a.max_n; // [slot][0 lo, 1 hi, 2 best key]
  __shared__ int bad;
  __shared__ int pair[16];

  if (tid == 0) bad = 0;
  if (tid < 16) pair[tid] = a.pair[tid];
  for (int s = tid; s < kFoldCtlSlots * 4; s += B) ctl[s] = (s % 4 == 0) ? INT32_MAX : -1;
  for (int s = tid; s < n; s += B) red[s] = E::kAccInit;
  __syncthreads();
  const uint8_t *src = a.x + a.off[sq];
  int mine = 0;
  for (int p = tid; p < n; p += B) {
    const uint8_t c = src[p];
    mine |= c > 3;
    xs[p] = c;
  }
  if (mine) atomicOr(&bad, 1);
  // span 0: F(i,i) = 0; every longer span starts as minus infinity when
  // cells can be left unevaluated (X-drop)
  if (XD)
    for (int e = tid; e < H * SC; e += B) G[e] = (T)E::kDead;
  __syncthreads();
  for (int p = tid; p < n; p += B) G[p] = (T)0; // span 0 (row 0, upper part)
  __syncthreads();
  if (bad || n <= 1) {
    if (tid == 0) {
      res->score = 0;
      res->i = 0;
      res->j = 0;
      res->full = (!bad && n == 1) ? 1 : 0;
      res->cells = 0;
      res->terms = 0;
      res->status = bad ? ALN_R_BAD_SYMBOL : ALN_R_OK;
      res->reserved = 0;
    }
    return;
  }

  int best = 0, bi = 0, bj = 0; // best cell through the last span (span 0: F = 0 at (0,0))
  int lo = 0, hi = n - 1;       // survivors of the last span
  long long cells = 0, terms = 0;
  int full = 0;
  const int X = a.xdrop;
  for (int t = 1; t < n; ++t) {
    const int ca = XD ? max(lo - 1, 0) : 0;
    const int cb = XD ? min(hi, n - 1 - t) : n - 1 - t;
    if (ca > cb) break;
    const int c = cb - ca + 1;
    cells += c;
    terms += (long long)c * t;
    const int slot = t % kFoldCtlSlots;
    int *cs = ctl + 4 * slot;
    const bool prune = XD && t > a.warmup;
    // survivors / best of this span; the slot two spans back is free again
    if (tid == 0) {
      int *nx = ctl + 4 * ((t + 1) % kFoldCtlSlots);
      nx[0] = INT32_MAX;
      nx[1] = -1;
      nx[2] = -1;
    }
    // this thread's survivors and best cell of the span, combined per wave
    // (DPP) and then per workgroup (one LDS atomic per wave)
    int my_lo = INT32_MAX, my_hi = -1, my_key = -1;
    // finish cell i of span t from its bifurcation maximum
    auto finish = [&](int i, int acc) {
      const int j = i + t;
      const int in = (t == 1) ? 0 : (int)G[fold_at<SC>(t - 2, i + 1, n, H)];
      const int s = (j - i > a.min_loop) ? pair[xs[i] * 4 + xs[j]] : 0;
      int v = max(acc, E::inner(in, s));
      bool keep = E::live(v);
      const int f = keep ? E::value(v) : 0;
      if (keep && prune && best - f > X) keep = false;
      G[fold_at<SC>(t, i, n, H)] = keep ? (T)f : (T)E::kDead;
      if (keep) {
        my_lo = min(my_lo, i);
        my_hi = max(my_hi, i);
        my_key = max(my_key, (f << 16) | (0xffff - i)); // highest F, then smallest i
      }
    };
    // 64 cells per wave; when fewer chunks than waves, each chunk's
    // u-range is cut into S = 2^ls pieces of len splits (shifts only: the
    // scalar unit, shared by the CU's waves, has no divide)
    const int chunks = (c + 63) >> 6;
    const int cl = chunks > 1 ? 32 - __builtin_clz(chunks - 1) : 0; // ceil(log2(chunks))
    const int ls = chunks >= W ? 0 : (31 - __builtin_clz(W)) - cl;
    const int S = 1 << ls;
    const int len = (t + S - 1) >> ls;
    int *rb = red;
    for (int item = wave; item < chunks * S; item += W) {
      const int ch = item >> ls, seg = item & (S - 1);
      const int u0 = min(seg * len, t), u1 = min(u0 + len, t);
      const int q = ch * 64 + lane;
      // lanes past the last cell read inside the triangle and drop the result
      const int i = ca + min(q, c - 1);
      const int acc = fold_partial<T, XD, SC>(G, n, H, t, i, u0, u1);
      if (q < c) {
        if (S == 1) finish(ca + q, acc);
        else atomicMax(&rb[q], acc);
      }
    }
    if (S > 1) {
      __syncthreads();
      for (int q = tid; q < c; q += B) {
        finish(ca + q, rb[q]);
        rb[q] = E::kAccInit; // ready for the next span (its atomics follow the barrier below)
      }
    }
    {
      const int wk = fold_wave_max(my_key);
      const int wl = XD ? fold_wave_min(my_lo) : 0;
      const int wh = XD ? fold_wave_max(my_hi) : 0;
      if (lane == 63 && wk >= 0) {
        if (XD) {
          atomicMin(&cs[0], wl);
          atomicMax(&cs[1], wh);
        }
        atomicMax(&cs[2], wk);
      }
    }
    __syncthreads();
    // every thread reads the span's outcome (the slot is not written again
    // before two more barriers)
    const int key = cs[2];
    if (key >= 0) {
      const int f = key >> 16, wi = 0xffff - (key & 0xffff);
      if (f >= best) { // a longer span wins ties
        best = f;
        bi = wi;
        bj = wi + t;
      }
    }
    if (XD) {
      if (key < 0) break; // nothing survived: the fold stops
      lo = cs[0];
      hi = cs[1];
    }
    if (t == n - 1) full = key >= 0;
  }
  if (tid == 0) {
    res->score = best;
    res->i = bi;
    res->j = bj;
    res->full = full;
    res->cells = cells;
    res->terms = terms;
    res->status = ALN_R_OK;
    res->reserved = 0;
  }
}


// ------------------------------------------------- unpruned, byte elements
// Every cell is live and every sum of two cells of one interval fits a byte (the
// planner bounds the scores by 253).  With intervals half open, G(i,j) = F(i,j-1),
// G(i,i) = 0, the recurrence is
//   G(i,j) = max( max over i < k < j of G(i,k) + G(k,j),
//                 G(i+1,j-1) + pair(x_i, x_{j-1}) ),
// a (max,+) closure of an upper triangle, so it runs by 16 x 16 tiles of bytes (256
// contiguous bytes each, tile rows packed): tile (I,J) first takes the products of
// the tiles (I,K) and (K,J), I < K < J, and is then completed by the terms that
// read itself and the diagonal tiles (I,I) and (J,J).  The tiles of one tile
// diagonal are independent: 2 barriers per 16 spans.
//
// Product of two tiles, one wavefront: a lane holds 4 rows x 4 columns and a quarter
// of the splits k; four k are four dwords of each operand, 16 byte splats and, per
// row and k, one 32-bit add of four sums and byte maxima by packed 16-bit ones
// (an odd byte is the high half of its 16 bits, whose low half only breaks
// ties; an even one is masked out first): 80 instructions and 8 LDS reads for 4096
// terms.  Swaps of half and quarter waves join the four quarters.  The products of
// a tile diagonal are cut evenly over the wavefronts, in tile order: a wavefront's
// first tile may have begun in another one, then its maxima go to a buffer
// of its own, which the completion joins.
//
// Completion, 16 lanes a tile (four tiles a wavefront), lane ii = row ii, 31 steps:
// at step d lane ii is at column jj = d - 15 + ii, so j - i is the same for all.
// The lane keeps its row's last 15 cells, nearest first, in four dwords, meets them
// with column jj of the diagonal tile (J,J) (kept transposed and in that order), and
// takes from lane ii + 1 the column's cells below its own, in the same order, and
// meets them with row ii of (I,I), fixed.  Cells not there are 0, which no term that
// counts is below.  Nothing on the chain from step to step goes through LDS.
//
// What bounds it: vector instructions (0.73 a cycle and CU at 496 nt, one workgroup a CU;
// 0.81 at 367 nt, two; 60% of them in products of bytes), with products on the matrix
// cores (0.52 and 0.55) the completions: 31 steps of about 56 instructions a tile diagonal, in which one
// workgroup a CU leaves SIMDs idle.  2 048 sequences, ms, before (a cell a lane and a
// barrier or two each span, a term two byte reads from LDS) / products of bytes / matrix
// cores: 76..500 nt 5.11 / 1.15 / 0.96, 400..500 nt 9.30 / 2.49 / 1.96, 40..127 nt
// 0.232 / 0.071 / 0.074; 4 of 400..500 nt 1.38 / 0.37 / 0.28.
using u16x2 = unsigned short __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t x, uint32_t y) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, x),
                                                                __builtin_bit_cast(u16x2, y)));
}
constexpr uint32_t kEven = 0x00ff00ffu;
// byte maxima of two dwords
__device__ __forceinline__ uint32_t max_u8x4(uint32_t x, uint32_t y) {
  return (pk_max_u16(x, y) & ~kEven) | pk_max_u16(x & kEven, y & kEven);
}

// This lane's parts of one pair of tiles: four rows by four splits, four splits by four columns.
struct FoldPair {
  uint32_t x[4], y[4];
  __device__ __forceinline__ void load(const uint8_t *a, const uint8_t *b) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      x[r] = *reinterpret_cast<const uint32_t *>(a + 16 * r);
      y[r] = *reinterpret_cast<const uint32_t *>(b + 16 * r);
    }
  }
  __device__ __forceinline__ void join(uint32_t (&e)[4], uint32_t (&o)[4]) const {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t s = __builtin_amdgcn_perm(x[r], x[r], 0x01010101u * k) + y[k];
        o[r] = pk_max_u16(o[r], s);
        e[r] = pk_max_u16(e[r], s & kEven);
      }
  }
};

// Pair scores of 0 and 1: on the matrix cores.  G(i,k) grows by 0 or 1 with each base,
// so within a tile row A(i,k) - A(i,0) and within a tile column B(k,j) - B(15,j) are
// 0..15, and 2 ^ (8 x) of them is a bf16 number; their product over k is a sum of at
// most 16 powers 2 ^ (8 (a + b)), whose exponent's multiple of 8 is the maximum, 0..30
// (a float's exponent field holds 8 x 30 + 4; a maximum of 0 may be flushed to
// zero, which reads the same).  Exact, and 4096 terms take one instruction and 20-odd
// to feed it.  The first operand is B transposed, so that a lane's result is the dword
// of row lane & 15, columns 4 (lane >> 4) ...
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
struct FoldUnitPair {
  uint32_t x, rb4;      // A(i, 4 kg ..), B(15, 4 kg ..)
  uint16_t ra, rb;      // A(i, 0), B(15, j)
  uint8_t y[4];         // B(4 kg .., j)
  __device__ __forceinline__ void load(const uint8_t *a, const uint8_t *b, int lane) {
    const int l = lane & 15, kg = lane >> 4;
    x = *reinterpret_cast<const uint32_t *>(a + 16 * l + 4 * kg);
    ra = a[16 * l];
    rb = b[240 + l];
    rb4 = *reinterpret_cast<const uint32_t *>(b + 240 + 4 * kg);
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = b[64 * kg + 16 * r + l];
  }
  __device__ __forceinline__ void join(uint32_t &e, uint32_t &o) const {
    const u16x2 scale = {1024, 1024}; // 8 << 7, a bf16 exponent of 8
    auto power = [&](uint32_t pair, uint16_t base, int bias) __attribute__((always_inline)) {
      const uint16_t c = (uint16_t)(bias * 128 - base * 1024);
      const u16x2 cc = {c, c};
      return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, pair) * scale + cc));
    };
    const uint32_t y01 = y[0] | ((uint32_t)y[1] << 16), y23 = y[2] | ((uint32_t)y[3] << 16);
    const uint2 av = make_uint2(power(__builtin_amdgcn_perm(0u, x, 0x0c010c00u), ra, 64),
                                power(__builtin_amdgcn_perm(0u, x, 0x0c030c02u), ra, 64));
    const uint2 bv = make_uint2(power(y01, rb, 63), power(y23, rb, 63));
    const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
        __builtin_bit_cast(s16x4, bv), __builtin_bit_cast(s16x4, av), f32x4{0, 0, 0, 0}, 0, 0, 0);
    const uint32_t hi = __builtin_amdgcn_perm(__float_as_uint(d[1]), __float_as_uint(d[0]), 0x0c0c0703u) |
                        __builtin_amdgcn_perm(__float_as_uint(d[3]), __float_as_uint(d[2]), 0x07030c0cu);
    const uint32_t v = ((hi >> 2) & 0x3f3f3f3fu) + rb4 + __builtin_amdgcn_perm(0u, (uint32_t)ra, 0u);
    o = pk_max_u16(o, v);
    e = pk_max_u16(e, v & kEven);
  }
};
// Products of cnt >= 1 tile pairs for one tile, from the first two on (bstep as below): the
// dword of row lane & 15, columns 4 (lane >> 4) ... of the joined tile.
__device__ __forceinline__ uint32_t fold_unit_products(const uint8_t *a, const uint8_t *b, int bstep,
                                                       int cnt, int lane) {
  uint32_t e = 0, o = 0;
  FoldUnitPair p0, p1;
  p0.load(a, b, lane);
  for (;;) { // the next pair's reads are in flight meanwhile
    if (cnt > 1) p1.load(a + 256, b + 256 * bstep, lane);
    p0.join(e, o);
    if (cnt <= 1) break;
    a += 512;
    b += 256 * (2 * bstep - 1);
    bstep -= 2;
    if (cnt > 2) p0.load(a, b, lane);
    p1.join(e, o);
    cnt -= 2;
    if (cnt <= 0) break;
  }
  return (o & ~kEven) | e;
}

// Products of cnt >= 1 tile pairs for one tile: a, b this lane's parts of the first two,
// bstep tiles from b's to the next, one less each time.  Returns the lane's dword of the
// joined tile: row 4 p + r, columns 4 q .. 4 q + 3 (p, q, and r by its quarter wave).
__device__ __forceinline__ uint32_t fold_products(const uint8_t *a, const uint8_t *b, int bstep,
                                                  int cnt) {
  uint32_t e[4] = {0, 0, 0, 0}, o[4] = {0, 0, 0, 0};
  FoldPair p0, p1;
  p0.load(a, b);
  for (;;) { // the next pair's reads are in flight meanwhile
    if (cnt > 1) p1.load(a + 256, b + 256 * bstep);
    p0.join(e, o);
    if (cnt <= 1) break;
    a += 512;
    b += 256 * (2 * bstep - 1);
    bstep -= 2;
    if (cnt > 2) p0.load(a, b);
    p1.join(e, o);
    cnt -= 2;
    if (cnt <= 0) break;
  }
  auto join32 = [](uint32_t u, uint32_t v) __attribute__((always_inline)) {
    const auto t = __builtin_amdgcn_permlane32_swap(u, v, false, false);
    return pk_max_u16(t[0], t[1]);
  };
  auto join16 = [](uint32_t u, uint32_t v) __attribute__((always_inline)) {
    const auto t = __builtin_amdgcn_permlane16_swap(u, v, false, false);
    return pk_max_u16(t[0], t[1]);
  };
  const uint32_t eo = join16(join32(e[0], e[1]), join32(e[2], e[3]));
  const uint32_t oo = join16(join32(o[0], o[1]), join32(o[2], o[3]));
  return (oo & ~kEven) | eo;
}

template <int W, bool UNIT>
__global__ __launch_bounds__(64 * W) void fold_tile_kernel(FoldArgs args) {
  constexpr int B = 64 * W;
  extern __shared__ __align__(16) uint8_t smem[];
  const FoldTask tk = args.tasks[blockIdx.x];
  const int n = tk.n;
  aln_fold_result *res = args.res + tk.seq;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  // LDS: tiles | transposed diagonal tiles | the wavefronts' partial tiles | 8 x codes
  const int NB = fold_tile_rows(n);
  uint8_t *G = smem;
  uint8_t *dT = G + fold_tile_rows(args.max_n) * (fold_tile_rows(args.max_n) + 1) / 2 * 256;
  uint8_t *part = dT + fold_tile_rows(args.max_n) * 256;
  uint8_t *xs = part + W * 256;
  __shared__ int bad;
  __shared__ uint32_t tab[4]; // pair scores of one base with the four
  if (tid == 0) bad = 0;
  if (tid < 4)
    tab[tid] = (uint32_t)args.pair[4 * tid] | ((uint32_t)args.pair[4 * tid + 1] << 8) |
               ((uint32_t)args.pair[4 * tid + 2] << 16) | ((uint32_t)args.pair[4 * tid + 3] << 24);
  __syncthreads();
  const uint8_t *src = args.x + args.off[tk.seq];
  int mine = 0;
  for (int p = tid; p < 16 * NB + 32; p += B) {
    const uint8_t c = p < n ? src[p] : 0;
    mine |= c > 3;
    xs[p] = c << 3;
  }
  if (mine) atomicOr(&bad, 1);
  // diagonal tiles and their transposes; tiles (I, I + 1) have no products
  for (int p = tid; p < 16 * NB; p += B) {
    const int I = p >> 4, r = 16 * (p & 15);
    *reinterpret_cast<uint4 *>(G + fold_tile_at(I, I, NB) + r) = make_uint4(0, 0, 0, 0);
    *reinterpret_cast<uint4 *>(dT + 256 * I + r) = make_uint4(0, 0, 0, 0);
    if (I + 1 < NB)
      *reinterpret_cast<uint4 *>(G + fold_tile_at(I, I + 1, NB) + r) = make_uint4(0, 0, 0, 0);
  }
  __syncthreads();
  if (bad || n <= 1) {
    if (tid == 0) {
      res->score = 0;
      res->i = 0;
      res->j = 0;
      res->full = (!bad && n == 1) ? 1 : 0;
      res->cells = 0;
      res->terms = 0;
      res->status = bad ? ALN_R_BAD_SYMBOL : ALN_R_OK;
      res->reserved = 0;
    }
    return;
  }
  const int ii = lane & 15, sub = lane >> 4;

  // diagonal tiles, a cell a lane and span
  for (int I = wave * 4 + sub; I < NB; I += W * 4) {
    uint8_t *T = G + fold_tile_at(I, I, NB), *D = dT + 256 * I;
    const uint8_t *xi = xs + 16 * I + ii;
    for (int t = 2; t < 16; ++t) {
      if (ii + t < 16) {
        int v = T[17 * ii + t + 15]; // (ii + 1, ii + t - 1)
        if (t - 1 > args.min_loop) v += (int)((tab[xi[0] >> 3] >> xi[t - 1]) & 255u);
        for (int u = 1; u < t; ++u)
          v = max(v, (int)T[17 * ii + u] + (int)D[16 * (ii + t) + t - u - 1]);
        T[17 * ii + t] = (uint8_t)v;
        D[16 * (ii + t) + t - 1] = (uint8_t)v;
      }
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    }
  }
  __syncthreads();

  for (int D = 1; D < NB; ++D) {
    const int c = NB - D, per = D - 1, units = c * per;
    if (per > 0) {
      int u = wave * units / W;
      const int u1 = (wave + 1) * units / W;
      if (u < u1) {
        int I = u / per, kk = u - I * per;
        const int p = (lane >> 2) & 3, q = lane & 3;
        const int aoff = 64 * p + 4 * sub, boff = 64 * sub + 4 * q;
        const int r = ((sub & 1) << 1) | (sub >> 1); // the row the swaps leave here
        const int dst = UNIT ? 16 * ii + 4 * sub : 16 * (4 * p + r) + 4 * q;
        while (u < u1) {
          const int cnt = min(per - kk, u1 - u), K = I + 1 + kk;
          const uint8_t *A = G + fold_tile_at(I, K, NB), *B = G + fold_tile_at(K, I + D, NB);
          const uint32_t v = UNIT ? fold_unit_products(A, B, NB - K - 1, cnt, lane)
                                  : fold_products(A + aoff, B + boff, NB - K - 1, cnt);
          uint8_t *to = kk ? part + 256 * wave : G + fold_tile_at(I, I + D, NB);
          *reinterpret_cast<uint32_t *>(to + dst) = v;
          u += cnt;
          ++I;
          kk = 0;
        }
      }
      __syncthreads();
    }
    for (int first = wave * 4; first < c; first += 4 * W) {
      const int I = min(first + sub, c - 1), J = I + D; // past the last: that one again
      uint8_t *T = G + fold_tile_at(I, J, NB) + 16 * ii;
      if (per > 0) { // wavefronts that began inside this tile's products
        const int from = I * per, to = from + per;
        uint4 m = *reinterpret_cast<const uint4 *>(T);
        bool more = false;
        for (int w = I * W / c + 1; w < W; ++w) {
          const int s = w * units / W;
          if (s >= to) break;
          if (s > from && (w + 1) * units / W > s) {
            const uint4 v = *reinterpret_cast<const uint4 *>(part + 256 * w + 16 * ii);
            m.x = max_u8x4(m.x, v.x);
            m.y = max_u8x4(m.y, v.y);
            m.z = max_u8x4(m.z, v.z);
            m.w = max_u8x4(m.w, v.w);
            more = true;
          }
        }
        if (more) *reinterpret_cast<uint4 *>(T) = m;
      }
      // row ii of (I,I) from column ii + 1 (then the next row's zeros)
      uint32_t g[4] = {0, 0, 0, 0};
      if (ii < 15) __builtin_memcpy(g, G + fold_tile_at(I, I, NB) + 17 * ii + 1, 16);
      const uint8_t *dt = dT + 256 * J + 16 * (ii - 15);
      uint8_t *cell = T + ii - 15;
      const uint8_t *xj = xs + 16 * J + ii - 16;
      const uint8_t *top = G + fold_tile_at(I + 1, J, NB) - 1;
      const uint32_t tabi = tab[xs[16 * I + ii] >> 3];
      const uint32_t left = G[fold_tile_at(I, J - 1, NB) + 16 * ii + 15];
      uint32_t corner = 0;
      if (D > 1) corner = G[fold_tile_at(I + 1, J - 1, NB) + 15];
      const int paired = min(args.min_loop, 4096) + 16 - 16 * D; // pairs from the step after this one
      uint32_t row[4] = {0, 0, 0, 0}, col[4] = {0, 0, 0, 0};
      uint32_t in1 = left, in2 = left; // last and last but one step's cells, or the one left of the tile
      struct Ahead {
        uint4 dt;
        uint32_t cell, xj, top;
      } ah[2];
      auto fetch = [&](int d) __attribute__((always_inline)) {
        Ahead f;
        f.dt = *reinterpret_cast<const uint4 *>(dt + 16 * d);
        f.cell = cell[d];
        f.xj = xj[d];
        f.top = d > 0 && d < 16 ? top[d] : 0;
        return f;
      };
      ah[0] = fetch(0);
      ah[1] = fetch(1);
#pragma unroll
      for (int d = 0; d < 31; ++d) {
        const Ahead f = ah[d & 1];
        if (d + 2 < 31) ah[d & 1] = fetch(d + 2);
        // the interval inside, plus the pair
        uint32_t in = (uint32_t)__builtin_amdgcn_update_dpp((int)(d ? f.top : corner), (int)in2,
                                                            0x101, 0xf, 0xf, false); // row_shl:1
        in += __builtin_amdgcn_ubfe(tabi, f.xj, d > paired ? 8 : 0);
        uint32_t v = max(f.cell, in);
        const int nd = min(4, (d + 3) / 4); // dwords that can hold cells by now
        if (nd) {
          const uint32_t dtw[4] = {f.dt.x, f.dt.y, f.dt.z, f.dt.w};
          uint32_t e = 0, o = 0;
#pragma unroll
          for (int k = 3; k >= 0; --k) // the newest cells are in the first
            if (k < nd) {
              const uint32_t s1 = row[k] + dtw[k], s2 = col[k] + g[k];
              o = pk_max_u16(o, pk_max_u16(s1, s2));
              e = pk_max_u16(e, pk_max_u16(s1 & kEven, s2 & kEven));
            }
          e = pk_max_u16(e, (o >> 8) & kEven);
          v = max(max(v, e >> 16), e & 0xffffu);
        }
        in2 = in1;
        in1 = v;
        if (d < 15) {
          const bool inside = ii >= 15 - d;
          in1 = inside ? v : left;
          v = inside ? v : 0u;
          if (inside) cell[d] = (uint8_t)v;
        } else if (d == 15 || ii <= 30 - d) {
          cell[d] = (uint8_t)v;
        }
#pragma unroll
        for (int k = 3; k > 0; --k) {
          row[k] = __builtin_amdgcn_alignbyte(row[k], row[k - 1], 3);
          col[k] = __builtin_amdgcn_alignbyte(col[k], col[k - 1], 3);
        }
        row[0] = (row[0] << 8) | v;
        col[0] = (col[0] << 8) | v;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (k <= (d >> 2)) // lane 15 takes none
            col[k] = (uint32_t)__builtin_amdgcn_mov_dpp((int)col[k], 0x101, 0xf, 0xf, true);
      }
    }
    __syncthreads();
  }
  if (tid == 0) { // every cell evaluated and kept, so the whole sequence is the best interval
    res->score = (int)G[fold_tile_at(0, n >> 4, NB) + (n & 15)];
    res->i = 0;
    res->j = n - 1;
    res->full = 1;
    res->cells = (int64_t)n * (n - 1) / 2;
    res->terms = (int64_t)(n - 1) * n * (n + 1) / 6;
    res->status = ALN_R_OK;
    res->reserved = 0;
  }
}

template <typename K>
static hipError_t launch_fold_lds(K kern, int block, size_t lds, const FoldArgs &a, hipStream_t s) {
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(a.ntasks), dim3(block), lds, s, a);
  return hipGetLastError();
}

template <typename T, bool XD, int B>
static hipError_t launch_fold_s(int stride, const FoldArgs &a, hipStream_t s) {
  const size_t lds = fold_lds_bytes(sizeof(T), stride, a.max_n);
  switch (stride) {
  case 128: return launch_fold_lds(fold_kernel<T, XD, B, 128>, B, lds, a, s);
  case 256: return launch_fold_lds(fold_kernel<T, XD, B, 256>, B, lds, a, s);
  case 384: return launch_fold_lds(fold_kernel<T, XD, B, 384>, B, lds, a, s);
  case 512: return launch_fold_lds(fold_kernel<T, XD, B, 512>, B, lds, a, s);
  default: return hipErrorInvalidValue;
  }
}

template <typename T, bool XD>
static hipError_t launch_fold_b(int block, int stride, const FoldArgs &a, hipStream_t s) {
  switch (block) {
  case 256: return launch_fold_s<T, XD, 256>(stride, a, s);
  case 512: return launch_fold_s<T, XD, 512>(stride, a, s);
  case 1024: return launch_fold_s<T, XD, 1024>(stride, a, s);
  default: return hipErrorInvalidValue;
  }
}

template <bool UNIT>
static hipError_t launch_fold_tiles(int block, const FoldArgs &a, hipStream_t s) {
  const size_t lds = fold_tile_lds_bytes(a.max_n, block / 64);
  switch (block) {
  case 256: return launch_fold_lds(fold_tile_kernel<4, UNIT>, block, lds, a, s);
  case 512: return launch_fold_lds(fold_tile_kernel<8, UNIT>, block, lds, a, s);
  case 1024: return launch_fold_lds(fold_tile_kernel<16, UNIT>, block, lds, a, s);
  default: return hipErrorInvalidValue;
  }
}

hipError_t launch_fold(int elt_bytes, int block, int stride, const FoldArgs &a, hipStream_t s) {
  if (a.ntasks <= 0) return hipSuccess;
  if (a.max_n + 1 > stride) return hipErrorInvalidValue;
  const bool xd = a.xdrop >= 0;
  if (elt_bytes == 2)
    return xd ? launch_fold_b<int16_t, true>(block, stride, a, s)
              : launch_fold_b<int16_t, false>(block, stride, a, s);
  if (elt_bytes == 1)
    return xd ? launch_fold_b<uint8_t, true>(block, stride, a, s)
              : (*std::max_element(a.pair, a.pair + 16) <= 1 ? launch_fold_tiles<true>(block, a, s)
                                                             : launch_fold_tiles<false>(block, a, s));
  return hipErrorInvalidValue;
}

} // namespace alnk
