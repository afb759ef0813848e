// aln_api.cpp -- host runtime behind include/aln.h.
//
// Planning happens on the host from the pairs' lengths: each pair gets a
// kernel and a tile shape, pairs of one shape are ordered longest first
// (largest cell count first, so the tail of a launch is short work), and the
// workspace is laid out as [task lists | traceback codes].  Executing a plan
// uploads the task lists from pinned memory and enqueues the kernels on the
// caller's stream; nothing is allocated on that path.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <functional>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "internal.h"
#include "runtime.h"

using alnk::DevScoring;
using alnk::PairTask;
using namespace alnrt;


namespace {


#define HIP_TRY(ctx, call)                                                       \
  do {                                                                           \
    hipError_t e_ = (call);                                                      \
    if (e_ != hipSuccess)                                                        \
      return fail((ctx), ALN_E_DEVICE, "%s failed: %s", #call, hipGetErrorString(e_)); \
  } while (0)

// Rows per lane for the strip kernel: fewest padded cells plus a per-step
// overhead of about eight cells per lane.
int choose_strip_rows(int32_t M, int32_t N) {
  if (M <= 512) return 8; // one strip: the fewest rows
  static const int cand[] = {8, 16, 24, 32};
  int best = 16;
  double best_cost = 1e300;
  for (int R : cand) {
    const int64_t HS = 64LL * R;
    const int64_t ns = (M + HS - 1) / HS;
    const double cost = (double)ns * (double)(N + 63) * 64.0 * (double)(R + 8);
    if (cost < best_cost) {
      best_cost = cost;
      best = R;
    }
  }
  return best;
}

hipEvent_t pool_event(aln_ctx *ctx) {
  if (!ctx->event_pool.empty()) {
    hipEvent_t e = ctx->event_pool.back();
    ctx->event_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Run `launch` (which enqueues one kernel on `st`); with profiling on, the
// launch is bracketed by events recorded on the same stream.
template <class F>
hipError_t timed_launch(aln_ctx *ctx, const char *name, hipStream_t st, F &&launch) {
  if (!ctx->profiling) return launch();
  hipEvent_t a = pool_event(ctx), b = pool_event(ctx);
  if (!a || !b) return hipErrorOutOfMemory;
  (void)hipEventRecord(a, st);
  hipError_t e = launch();
  (void)hipEventRecord(b, st);
  ctx->timed.push_back({name, a, b});
  return e;
}

} // namespace

aln_status alnrt::fail(aln_ctx *ctx, aln_status st, const char *fmt, ...) {
  if (ctx) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    ctx->err = buf;
  }
  return st;
}

extern "C" {

int32_t aln_abi_version(void) { return ALN_ABI_VERSION; }

aln_status aln_create(aln_ctx **ctx, int32_t device) {
  if (!ctx) return ALN_E_INVAL;
  *ctx = nullptr;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || device < 0 || device >= count)
    return ALN_E_DEVICE;
  if (hipSetDevice(device) != hipSuccess) return ALN_E_DEVICE;
  aln_ctx *c = new (std::nothrow) aln_ctx;
  if (!c) return ALN_E_NOMEM;
  c->device = device;
  int v = 0;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && v > 0)
    c->cus = v;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, device) ==
          hipSuccess && v > 0)
    c->lds_per_cu = v;
  if (alnrt::scratch_init(c) != ALN_OK) {
    delete c;
    return ALN_E_DEVICE;
  }
  *ctx = c;
  return ALN_OK;
}

aln_status aln_create_host(aln_ctx **ctx, int32_t cus, int32_t lds_per_cu) {
  if (!ctx || cus < 0 || lds_per_cu < 0) return ALN_E_INVAL;
  *ctx = nullptr;
  aln_ctx *c = new (std::nothrow) aln_ctx;
  if (!c) return ALN_E_NOMEM;
  c->device = -1;
  if (cus > 0) c->cus = cus;
  if (lds_per_cu > 0) c->lds_per_cu = lds_per_cu;
  *ctx = c;
  return ALN_OK;
}

void aln_destroy(aln_ctx *ctx) {
  if (!ctx) return;
  if (ctx->device < 0) {
    delete ctx;
    return;
  }
  (void)hipSetDevice(ctx->device);
  for (DevScoring *d : ctx->dsc) (void)hipFree(d);
  for (auto &t : ctx->timed) {
    (void)hipEventDestroy(t.a);
    (void)hipEventDestroy(t.b);
  }
  for (hipEvent_t e : ctx->event_pool) (void)hipEventDestroy(e);
  delete ctx;
}

aln_status aln_set_profiling(aln_ctx *ctx, int32_t enable) {
  if (!ctx) return ALN_E_INVAL;
  ctx->profiling = enable != 0;
  return ALN_OK;
}

int32_t aln_kernel_times(aln_ctx *ctx, const char **names, double *ms, int64_t *launches,
                         int32_t max) {
  if (!ctx || max < 0 || (max > 0 && (!names || !ms || !launches))) return ALN_E_INVAL;
  (void)hipSetDevice(ctx->device);
  int32_t nout = 0;
  for (auto &t : ctx->timed) {
    float el = 0.f;
    (void)hipEventSynchronize(t.b);
    (void)hipEventElapsedTime(&el, t.a, t.b);
    int32_t k = 0;
    while (k < nout && strcmp(names[k], t.name) != 0) ++k;
    if (k == nout) {
      if (nout == max) continue;
      names[nout] = t.name;
      ms[nout] = 0.0;
      launches[nout] = 0;
      ++nout;
    }
    ms[k] += el;
    launches[k] += 1;
    ctx->event_pool.push_back(t.a);
    ctx->event_pool.push_back(t.b);
  }
  ctx->timed.clear();
  return nout;
}

const char *aln_last_error(const aln_ctx *ctx) { return ctx ? ctx->err.c_str() : ""; }

aln_status aln_set_scoring(aln_ctx *ctx, const aln_scoring *sc, int32_t *scoring_id) {
  if (!ctx || !sc || !scoring_id || !sc->matrix) return fail(ctx, ALN_E_INVAL, "null argument");
  const int A = sc->alphabet;
  if (A < 1 || A > alnk::kMaxAlphabet)
    return fail(ctx, ALN_E_INVAL, "alphabet %d outside 1..%d", A, alnk::kMaxAlphabet);
  if (sc->gap_open > 0 || sc->gap_extend > 0 || sc->gap_open < -1024 || sc->gap_extend < -1024)
    return fail(ctx, ALN_E_INVAL, "gap penalties must lie in [-1024, 0]");
  DevScoring h;
  memset(&h, 0, sizeof h);
  h.alphabet = A;
  h.gap_open = sc->gap_open;
  h.gap_extend = sc->gap_extend;
  h.max_s = -(1 << 30);
  h.min_s = 1 << 30;
  bool mm = true;
  for (int a = 0; a < A; ++a)
    for (int b = 0; b < A; ++b) {
      const int v = sc->matrix[a * A + b];
      if (v < -127 || v > 127)
        return fail(ctx, ALN_E_INVAL, "substitution score %d outside [-127, 127]", v);
      h.mat[a * alnk::kMaxAlphabet + b] = v;
      h.max_s = std::max(h.max_s, v);
      h.min_s = std::min(h.min_s, v);
      const int ref = (a == b) ? sc->matrix[0] : (A > 1 ? sc->matrix[1] : 0);
      if (v != ref) mm = false;
    }
  h.match_mismatch = mm ? 1 : 0;
  h.match = sc->matrix[0];
  h.mismatch = A > 1 ? sc->matrix[1] : 0;
  for (int a = 0; a < A; ++a) {
    uint32_t w = 0;
    for (int b = 0; b < 4; ++b) {
      const int v = (b < A) ? h.mat[a * alnk::kMaxAlphabet + b] : -128;
      w |= ((uint32_t)(v & 0xff)) << (8 * b);
    }
    h.rowtab[a] = w;
  }
  if (ctx->device < 0) { // no device: the host mirror only
    ctx->dsc.push_back(nullptr);
    ctx->hsc.push_back(h);
    *scoring_id = (int32_t)ctx->dsc.size() - 1;
    return ALN_OK;
  }
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  DevScoring *d = nullptr;
  HIP_TRY(ctx, hipMalloc(&d, sizeof(DevScoring)));
  hipError_t e = hipMemcpy(d, &h, sizeof h, hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(d);
    return fail(ctx, ALN_E_DEVICE, "hipMemcpy scoring: %s", hipGetErrorString(e));
  }
  ctx->dsc.push_back(d);
  ctx->hsc.push_back(h);
  *scoring_id = (int32_t)ctx->dsc.size() - 1;
  return ALN_OK;
}

} // extern "C"

// Pairs from which bands below 256 diagonals leave the antidiagonal kernel (and one-strip
// pairs share a launch with longer ones).  Strips are shorter from one pair on (with paths,
// w = 64, us, antidiagonals / strips: one pair of 300 rows 454 / 140, of 1 000 1 416 / 324, of
// 20 000 28 000 / 5 740; three 475 / 143, 1 490 / 334, 29 300 / 5 770): up to three pairs keep
// the kernel that plans of so few have always named.
constexpr int32_t kStripBandPairs = 4;
// Pairs from which rolling blocks are used.  (Four to fifteen run on strips: blocks of two
// rows would be shorter there too, 15 pairs of 5 000 rows, w = 64, 1.12 against 1.52 ms, blocks
// of four, for wider bands, longer, w = 100 1.65 against 1.53.)
constexpr int32_t kRollPairs = 16;

// Rolling blocks for a band: rows a block and lanes a pair, 0 where none fits.
// Two rows a block take fewest instructions a row (78, four 112) and so the
// least time for a pair alone; on 16 lanes four pairs share them, which a band
// of up to 15 cells either side allows.  Four rows on 16 lanes allow twice
// that, once the pairs outnumber two wavefronts a SIMD.
static void roll_shape(const aln_ctx *ctx, int64_t n, int32_t M, int32_t N, int32_t w, int *rows,
                       int *lanes) {
  *rows = *lanes = 0;
  const bool many = n > 2LL * 4 * ctx->cus;
  static const int shapes[4][2] = {{2, 16}, {4, 16}, {2, 64}, {4, 64}};
  for (const auto &sh : shapes) {
    if (sh[0] == 4 && sh[1] == 16 && !many) continue;
    if (alnk::roll_fits(M, N, w, sh[0], sh[1])) {
      *rows = sh[0];
      *lanes = sh[1];
      return;
    }
  }
}

// Lanes a side for n X-drop sides of a 64-cell window.  Four lanes of sixteen
// cells take the fewest instructions a cell (240 a step for sixteen sides, 150
// for eight, 110 for four), but a step's instructions are also what the longest
// side waits for, and a small batch is no longer than that.  So four only once
// their wavefronts fill four slots a SIMD, sixteen while theirs take at most
// four.  Measured, sides of 150..5 000 bp, X = 100, 16 / 8 / 4 lanes in ms:
// 4 000 sides 4.7 / 5.6 / 8.0 (with codes 7.1 / 8.7 / 12.5), 12 000 6.2 / 6.3 /
// 8.5 (9.0 / 10.0 / 15), 25 000 9.6 / 8.6 / 11.3 (12.4 / 12.3 / 16), 50 000
// 15.8 / 12.5 / 13.6 (20.8 / 17.6 / 19.1), 100 000 29.0 / 20.2 / 18.4.
static int lanes_per_side(const aln_ctx *ctx, int64_t n) {
  const int64_t simds = 4LL * ctx->cus;
  return n <= 16 * simds ? 16 : (n <= 64 * simds ? 8 : 4);
}

// Z-drop sides from which the lanes form (eight lanes, a window of 128 cells)
// replaces one wavefront a side.  Sides of 150..5 000 bp at Z = 100, the first launch of
// each form in ms, one a wavefront / lanes: 4 000 sides 5.2 / 11.0, 12 000 9.6 / 11.0,
// 16 384 12.8 / 12.9, 20 000 15.3 / 14.4, 40 000 29.5 / 19.5.
static int64_t zdrop_lanes_from(const aln_ctx *ctx) { return 16LL * 4 * ctx->cus + 1; }

// Whether a Z-drop region stays within d diagonals either side of the best cell's: a gap
// of L costs |o| + L |e| and is forgiven L, so it reaches about (Z - |o|) / (|e| - 1) (at
// e = -1 any).
static bool zdrop_within(const DevScoring &sc, const aln_params &p, int64_t d) {
  return sc.gap_extend < -1 && (int64_t)p.xdrop + sc.gap_open <= d * (-sc.gap_extend - 1);
}
// d of what counts on few regions past 512 diagonals, the lanes form and the widening pass
// over them: the longer the sides, the further the widest regions go past the estimate, so
// that they outgrow 512 from d = 235 on at 2 500 bp and from 205 at 6 000, not yet at 180
// and 20 000.
constexpr int kZdropReach = 180;

// Interior cells (1 <= i <= M, 1 <= j <= N) of the static band: row i keeps
// floor(iN/M) - w <= j <= floor(iN/M) + w.  Rows whose band is clipped by
// column 1 or column N are counted one by one (the centre floor(iN/M) is
// non-decreasing in i, so they form a prefix and a suffix of the rows); every
// other row holds 2w + 1 cells.
static int64_t band_cells(int64_t M, int64_t N, int64_t w) {
  if (M <= 0 || N <= 0) return 0;
  if (w >= std::max(M, N)) return M * N;
  auto centre = [&](int64_t i) { return i * N / M; };
  auto row = [&](int64_t i) {
    const int64_t lo = std::max<int64_t>(1, centre(i) - w), hi = std::min(N, centre(i) + w);
    return hi >= lo ? hi - lo + 1 : 0;
  };
  // last row clipped on the left (centre <= w), first clipped on the right
  int64_t a = 0, lo = 1, hi = M;
  while (lo <= hi) {
    const int64_t mid = (lo + hi) / 2;
    if (centre(mid) <= w) { a = mid; lo = mid + 1; } else { hi = mid - 1; }
  }
  int64_t b = M + 1;
  lo = 1;
  hi = M;
  while (lo <= hi) {
    const int64_t mid = (lo + hi) / 2;
    if (centre(mid) + w > N) { b = mid; hi = mid - 1; } else { lo = mid + 1; }
  }
  int64_t total = 0;
  if (b <= a + 1) {
    for (int64_t i = 1; i <= M; ++i) total += row(i);
    return total;
  }
  for (int64_t i = 1; i <= a; ++i) total += row(i);
  for (int64_t i = b; i <= M; ++i) total += row(i);
  return total + (b - a - 1) * (2 * w + 1);
}

// Indices 0 .. key.size() - 1, largest key first, equal keys in index order.  By digits:
// a plan sorts its pairs on every batch, and a comparison sort of 100 000 took half of
// its time.
static std::vector<int32_t> order_desc(const std::vector<uint64_t> &key) {
  constexpr int kBits = 11, kDigits = 6; // 66 bits
  constexpr uint32_t kMask = (1u << kBits) - 1;
  const size_t n = key.size();
  std::vector<int32_t> at(n);
  std::iota(at.begin(), at.end(), 0);
  if (n < 512) {
    std::stable_sort(at.begin(), at.end(), [&](int32_t a, int32_t b) { return key[a] > key[b]; });
    return at;
  }
  std::vector<uint32_t> count((size_t)kDigits << kBits);
  for (const uint64_t k : key)
    for (int d = 0; d < kDigits; ++d) ++count[((size_t)d << kBits) + ((k >> (d * kBits)) & kMask)];
  std::vector<int32_t> to(n);
  for (int d = 0; d < kDigits; ++d) {
    uint32_t *const c = &count[(size_t)d << kBits];
    auto digit = [&](int32_t k) { return (uint32_t)(key[k] >> (d * kBits)) & kMask; };
    if (c[digit(0)] == n) continue; // the same in every key
    uint32_t sum = 0;
    for (int v = (int)kMask; v >= 0; --v) {
      const uint32_t here = c[v];
      c[v] = sum;
      sum += here;
    }
    for (const int32_t k : at) to[c[digit(k)]++] = k;
    at.swap(to);
  }
  return at;
}

aln_status alnrt::plan_build(aln_ctx *ctx, int32_t scoring_id, const aln_params *params, int32_t n,
                             const int32_t *q_len_host, const int32_t *r_len_host,
                             aln_plan **plan) {
  if (!ctx || !params || !plan || n < 0 || (n > 0 && (!q_len_host || !r_len_host)))
    return fail(ctx, ALN_E_INVAL, "null argument or negative n");
  *plan = nullptr;
  if (scoring_id < 0 || scoring_id >= (int32_t)ctx->dsc.size())
    return fail(ctx, ALN_E_INVAL, "unknown scoring id %d", scoring_id);
  const aln_params &p = *params;
  if (p.mode < ALN_GLOBAL || p.mode > ALN_EXTEND) return fail(ctx, ALN_E_INVAL, "bad mode");
  if (p.prune < ALN_FULL || p.prune > ALN_SEARCH) return fail(ctx, ALN_E_INVAL, "bad prune");
  if (p.prune == ALN_BAND && p.band_w < 0) return fail(ctx, ALN_E_INVAL, "band_w < 0");
  const bool dyn_prune = p.prune == ALN_XDROP || p.prune == ALN_ZDROP;
  if (dyn_prune && (p.xdrop < 0 || p.mode != ALN_EXTEND))
    return fail(ctx, ALN_E_INVAL, "XDROP / ZDROP need mode EXTEND and a threshold >= 0");
  if (p.width < ALN_W_AUTO || p.width > ALN_W_I32) return fail(ctx, ALN_E_INVAL, "bad width");
  const DevScoring &hs = ctx->hsc[scoring_id];
  const int64_t per_step = (int64_t)std::abs(hs.gap_open) + std::abs(hs.gap_extend) + 128;
  if (p.prune == ALN_SEARCH) {
    if (p.mode != ALN_GLOBAL || p.want_cigar)
      return fail(ctx, ALN_E_UNSUPPORTED, "SEARCH is GLOBAL, score only, without CIGAR");
    if (!hs.match_mismatch || hs.match != 0 || hs.mismatch >= 0 || hs.gap_open > 0 ||
        hs.gap_extend >= 0)
      return fail(ctx, ALN_E_UNSUPPORTED,
                  "SEARCH needs penalties: match 0, one mismatch score < 0, open <= 0, extend < 0");
  }

  aln_plan *pl = new (std::nothrow) aln_plan;
  if (!pl) return fail(ctx, ALN_E_NOMEM, "plan allocation");
  pl->ctx = ctx;
  pl->scoring_id = scoring_id;
  pl->p = p;
  pl->n = n;
  pl->qlen.assign(q_len_host, q_len_host + n);
  pl->rlen.assign(r_len_host, r_len_host + n);
  const bool small = hs.alphabet <= 4;

  int32_t maxM = 0, maxN = 0;
  for (int32_t i = 0; i < n; ++i) {
    maxM = std::max(maxM, pl->qlen[i]);
    maxN = std::max(maxN, pl->rlen[i]);
  }
  pl->max_m = maxM;
  pl->max_n = maxN;
  // score-major search: one workgroup per pair, longest first, both
  // sequences and the furthest-row arrays in LDS.  Unit edit costs: 1 to 8
  // wavefronts share a pair when two rows fit in LDS, else one wavefront
  // updates a single row in place.  Gap-affine penalties: 1 to 8 wavefronts
  // over rings of past H, E and F rows.
  if (p.prune == ALN_SEARCH) {
    std::vector<uint64_t> len(n);
    for (int32_t i = 0; i < n; ++i) len[i] = (uint64_t)pl->qlen[i] + (uint64_t)pl->rlen[i];
    const std::vector<int32_t> order = order_desc(len);
    LaunchDesc L{};
    L.kind = K_SEARCH;
    L.mode = ALN_GLOBAL;
    L.first = 0;
    L.count = n;
    L.lds_bnd = (int32_t)align_up((uint64_t)maxM + 20, 16);  // query codes + padding
    L.lds_prof = (int32_t)align_up((uint64_t)maxN + 20, 16); // reference codes + padding
    L.lds_f = (int32_t)align_up(((uint64_t)maxM + maxN + 1) * 2, 16); // int16 rows
    if (maxM > 32767 || (int64_t)L.lds_bnd + L.lds_prof + L.lds_f > 160 * 1024) {
      delete pl;
      return fail(ctx, ALN_E_UNSUPPORTED, "SEARCH needs M <= 32767 and the longest M plus the longest N of the batch <= about 54000");
    }
    L.waves = (int64_t)L.lds_bnd + L.lds_prof + 2 * (int64_t)L.lds_f <= 160 * 1024 ? 4 : 1;
    const bool unit = hs.mismatch == -1 && hs.gap_open == 0 && hs.gap_extend == -1;
    if (!unit) { // gap-affine: rings of past score rows, four wavefronts
      L.pen_x = -hs.mismatch;
      L.pen_o = -hs.gap_open;
      L.pen_e = -hs.gap_extend;
      L.ring_h = std::max(L.pen_x, L.pen_o + L.pen_e) + 1;
      L.ring_e = L.pen_e + 1;
      L.waves = 4;
      const int64_t lds = (int64_t)L.lds_bnd + L.lds_prof +
                          (int64_t)(L.ring_h + 2 * L.ring_e) * L.lds_f;
      if (lds > 160 * 1024) {
        delete pl;
        return fail(ctx, ALN_E_UNSUPPORTED,
                    "gap-affine SEARCH keeps %d score rows of %d bytes in LDS: %lld bytes > 160 KB",
                    L.ring_h + 2 * L.ring_e, L.lds_f, (long long)lds);
      }
      // First pass: rows of diagonals -dcap..dcap, dcap as large as lets four
      // workgroups share a CU; pairs whose range outgrows it run again with
      // full rows.  Skipped when capped rows would not be shorter.
      const int64_t nrows = L.ring_h + 2 * L.ring_e;
      const int64_t per_row = (40 * 1024 - (int64_t)L.lds_bnd - L.lds_prof) / nrows;
      const int64_t cap = (per_row / 2 - 1) / 2;
      if (cap >= 16 && 2 * cap + 1 < (int64_t)maxM + maxN + 1) {
        L.dcap = (int32_t)cap;
        L.lds_fc = (int32_t)align_up((uint64_t)(2 * cap + 1) * 2, 16);
        if ((int64_t)L.lds_bnd + L.lds_prof + nrows * L.lds_fc > 40 * 1024) { // rounding
          L.dcap -= 8;
          L.lds_fc = (int32_t)align_up((uint64_t)(2 * L.dcap + 1) * 2, 16);
        }
      }
      // Only multiples of the penalties' common divisor are scores, so the kernel
      // counts in it, over fewer rows (what fits and the cap above stay those of
      // the plain penalties).
      L.pen_g = std::gcd(L.pen_x, std::gcd(L.pen_o + L.pen_e, L.pen_e));
      L.pen_x /= L.pen_g;
      L.pen_o /= L.pen_g;
      L.pen_e /= L.pen_g;
      L.ring_h = std::max(L.pen_x, L.pen_o + L.pen_e) + 1;
      L.ring_e = L.pen_e + 1;
    }
    if (unit && L.waves == 4) {
      // A first pass with rows of the diagonals that a distance needs (of unrelated
      // sequences of four letters about half their length; at least the lengths'
      // difference), where LDS, and not the batch, limits the pairs a CU holds and it holds
      // few: 4 096 of 2 000 nt 163 -> 140 us, 1 000 of 7..8 knt 447 -> 354, the second
      // launch that looks for marked pairs included.  (Unrelated sequences of more letters
      // lie further apart, five 0.58 of their length, twenty 0.86: those pairs leave the
      // first pass early.)
      int32_t cap = (int32_t)(0.55 * std::max(maxM, maxN)) + 8;
      for (int32_t i = 0; i < n; ++i) cap = std::max(cap, std::abs(pl->qlen[i] - pl->rlen[i]) + 8);
      const int64_t full = (int64_t)L.lds_bnd + L.lds_prof + 2 * (int64_t)L.lds_f;
      const int64_t fit = 160 * 1024 / full;
      if (5LL * (2 * cap + 1) <= 4LL * (maxM + maxN + 1) && fit < 16 && n > ctx->cus * fit) {
        L.dcap = cap;
        L.lds_fc = (int32_t)align_up((uint64_t)(2 * cap + 1) * 2, 16);
      }
    }
    for (int32_t i : order) {
      PairTask t;
      memset(&t, 0, sizeof t);
      t.pair = i;
      t.tb_off = -1;
      pl->tasks.push_back(t);
    }
    pl->launches.push_back(L);
    pl->tasks_bytes = align_up(sizeof(PairTask) * std::max<size_t>(pl->tasks.size(), 1));
    pl->upload_bytes = sizeof(PairTask) * pl->tasks.size();
    pl->tb_base = pl->tasks_bytes;
    pl->tb_bytes = 0;
    pl->ws_bytes = pl->tasks_bytes;
    pl->cigar_words = 0;
    *plan = pl;
    return ALN_OK;
  }

  // packed int16 Smith-Waterman: LOCAL, full matrix, score + end cell
  const int rerun_rows = 16;
  const int32_t rerun_bnd = (int32_t)align_up((uint64_t)(maxN + 1) * 8, 16);
  const int32_t rerun_prof = small ? 0 : (int32_t)align_up((uint64_t)hs.alphabet * 64 * rerun_rows, 16);
  const bool use_sw16 = p.mode == ALN_LOCAL && p.prune == ALN_FULL && !p.want_cigar &&
                        p.width != ALN_W_I32 && n > 0 && hs.alphabet < alnk::kMaxAlphabet &&
                        maxN <= 65535 - 63 && maxM < (1 << 20) &&
                        4LL * (rerun_bnd + rerun_prof) <= 160 * 1024;
  if (use_sw16) {
    // rows per lane: forced while the autotuner measures, else the
    // ALN_SW16_ROWS override, else the autotuner's choice, else 16 or 8 (below)
    int tile = 0;
    if (ctx->tuning.valid) tile = ctx->tuning.sw16_rows;
    if (const char *ev = getenv("ALN_SW16_ROWS")) {
      const int r = atoi(ev);
      if (r == 4 || r == 8 || r == 12 || r == 16) tile = r;
    }
    if (ctx->force_sw16_rows) tile = ctx->force_sw16_rows;
    auto nstr = [](int32_t m, int32_t hs) { return (m + hs - 1) / hs; };
    // pairs sorted by the rows a lane of all their strips, then columns, longest
    // first; consecutive pairs share a task (the two 16-bit halves), so the halves
    // match
    struct TaskDim {
      int32_t pa, pb, mmax, nmax;
    };
    std::vector<TaskDim> td;
    auto make_tasks = [&](int32_t unit) {
      std::vector<uint64_t> key(n);
      for (int32_t i = 0; i < n; ++i)
        key[i] = ((uint64_t)nstr(pl->qlen[i], unit) << 32) | (uint32_t)pl->rlen[i];
      const std::vector<int32_t> order = order_desc(key);
      td.clear();
      td.reserve((size_t)(n + 1) / 2);
      for (int32_t q = 0; q < n; q += 2) {
        TaskDim t{order[q], q + 1 < n ? order[q + 1] : -1, pl->qlen[order[q]], pl->rlen[order[q]]};
        if (t.pb >= 0) {
          t.mmax = std::max(t.mmax, pl->qlen[t.pb]);
          t.nmax = std::max(t.nmax, pl->rlen[t.pb]);
        }
        td.push_back(t);
      }
    };
    struct Item {
      int64_t steps;      // its serial time
      int32_t first, end; // tasks
      int32_t wide;       // the one pair of a wide item, or -1; kBoth: its task's two
    };
    constexpr int32_t kBoth = -2;
    // What a task that runs wide becomes: nothing runs wide; two items, a pair on all lanes
    // each; one item, the two pairs in the halves of the lanes' words as on 16 lanes.
    enum Form { kNarrow, kWideOne, kWideBoth };
    struct Layout {
      int R = 0;
      Form form = kWideOne;
      std::vector<Item> items;
      double time = 0;    // estimate, instructions of one wavefront
      uint64_t bytes = 0; // boundary rows, all tasks narrow
    };
    const int pct_asked = ctx->force_sw16_wide_pct
                              ? ctx->force_sw16_wide_pct
                              : (ctx->tuning.valid ? ctx->tuning.sw16_wide_pct : 0);
    auto lay_out = [&](int R, Form form) {
      Layout o;
      o.R = R;
      o.form = form;
      const int32_t nt = (int32_t)td.size();
      // Serial column steps of one wavefront, in sixteenths of a step of R rows a lane
      // (the last strip's steps are shorter): a group of four tasks on 16-lane
      // groups runs the strips of the tallest over the widest reference (plus the
      // lane skew); a wide item runs one pair in 128*R-row strips, or two in 64*R-row ones.
      auto strips16 = [&](int32_t m, int32_t lanes) -> int64_t {
        const int32_t full = std::max(nstr(m, lanes * R) - 1, 0);
        const int32_t last = std::max(4, nstr(m - full * lanes * R, 4 * lanes) * 4);
        return 16 * full + 16 * (12 * last + 22) / (12 * R + 22);
      };
      auto narrow = [&](int32_t first, int32_t end) {
        int32_t m = 0, nm = 0;
        for (int32_t k = first; k < end; ++k) {
          m = std::max(m, td[k].mmax);
          nm = std::max(nm, td[k].nmax);
        }
        return strips16(m, 16) * (nm + 15);
      };
      // Load model: one wavefront per item; LDS bounds the wavefronts per CU.
      // A lone wavefront keeps its SIMD about 4/5 busy, so a second one on the
      // same SIMD adds about a quarter of a wavefront's rate.
      const size_t lds16 = alnk::sw16_lds_bytes(R, hs.alphabet);
      const int wpc = (int)std::max<size_t>(1, std::min<size_t>(16, (size_t)ctx->lds_per_cu / lds16));
      const double capacity =
          (double)ctx->cus * (std::min(wpc, 4) + 0.25 * std::min(std::max(wpc - 4, 0), 4));
      int64_t total = 0;
      for (int32_t k = 0; k < nt; k += 4) total += narrow(k, std::min(nt, k + 4));
      // A task whose own strips take longer than most of a wave slot's share
      // of the launch would finish last: it runs wide.
      const int wide_pct = pct_asked ? pct_asked : 80;
      const double wide_above = wide_pct < 0 || form == kNarrow
                                    ? 1e300
                                    : wide_pct / 100.0 * (double)total / capacity;
      // Narrow items hold up to four consecutive tasks that are not wide (a wide task
      // between them ends an item: the tallest come first, so there are few).
      int32_t open = -1;
      auto close = [&](int32_t end) {
        if (open >= 0) o.items.push_back(Item{narrow(open, end), open, end, -1});
        open = -1;
      };
      for (int32_t k = 0; k < nt; ++k) {
        if (nstr(td[k].mmax, 16 * R) > 1) o.bytes += align_up((uint64_t)(td[k].nmax + 1) * 8, 16);
        if ((double)narrow(k, k + 1) > wide_above) {
          close(k);
          if (form == kWideBoth)
            o.items.push_back(Item{strips16(td[k].mmax, 64) * (td[k].nmax + 63), k, k + 1, kBoth});
          else for (int32_t pair : {td[k].pa, td[k].pb})
            if (pair >= 0)
              o.items.push_back(Item{strips16(pl->qlen[pair], 128) * (pl->rlen[pair] + 127), k, k + 1,
                                     pair});
          continue;
        }
        if (open < 0) open = k;
        if (k + 1 - open == 4) close(k + 1);
      }
      close(nt);
      int64_t longest = 0, all = 0;
      for (const Item &it : o.items) {
        longest = std::max(longest, it.steps);
        all += it.steps;
      }
      o.time = std::max((double)longest, (double)all / capacity);
      // (few items a slot: of the (r - 1) slots + 1 longest, r share a slot)
      const size_t slots = (size_t)ctx->cus * std::min(wpc, 4);
      if (o.items.size() > slots && o.items.size() <= 4 * slots) {
        std::vector<int64_t> steps;
        for (const Item &it : o.items) steps.push_back(it.steps);
        for (size_t r = 2; (r - 1) * slots < steps.size(); ++r) {
          std::nth_element(steps.begin(), steps.begin() + (r - 1) * slots, steps.end(), std::greater<int64_t>());
          o.time = std::max(o.time, (double)r * (double)steps[(r - 1) * slots] * (double)slots / capacity);
        }
      }
      o.time *= (12 * R + 22) / 16.;
      return o;
    };
    // By the model's time.  A threshold in shares of a slot's load sends whole batches wide
    // where their items are about as many as the slots, and a launch of nothing but wide
    // items is bound by instructions: then four tasks a wavefront take the fewest, and two
    // pairs an item fewer than one (less skew, and more rows a lane).  Four letters, us, one
    // pair an item / none wide / the choice: 9 000 pairs of 210..300 letters 501 / 295 / 297,
    // 6 000 of 490..700 against 196..280 515 / 476 / 304 (two), 4 000 of 35..50 129 / 42 / 42.
    // A tuned threshold stands, and about a tie stays with one.
    auto best_of = [&](int R) {
      Layout b = lay_out(R, kWideOne);
      if (pct_asked < 0) return b;
      for (const Form f : {kWideBoth, kNarrow}) {
        if (f == kNarrow && pct_asked) continue;
        Layout o = lay_out(R, f);
        if (o.time < 0.96 * b.time) b = std::move(o);
      }
      return b;
    };
    make_tasks(64);
    Layout lay = best_of(tile ? tile : 16);
    if (!tile && alnk::sw16_lds_bytes(16, hs.alphabet) * 4 > (size_t)ctx->lds_per_cu) {
      // Profiles of 16 rows a lane leave SIMDs without a wavefront (19 letters and
      // more), ones of 8 rows take more instructions a cell: the shorter of the two, by
      // the model above.  20 letters, 16 / 8 rows, ms: 1 024 pairs of about 350 0.70 /
      // 0.78, 8 192 0.95 / 0.98, 16 384 1.53 / 1.21, 40 000 3.54 / 2.49; 30 000 of about
      // 120 0.39 / 0.33.  (Four letters, 20 000 reads of 150: 0.27 / 0.35, so always 16.)
      Layout small8 = best_of(8);
      if (small8.time < lay.time) lay = std::move(small8);
    }
    // More strips and a finer order may take more boundary rows than 16 rows a lane and an
    // order by strips: not past what a call without allocation has (the rest of the
    // workspace is less than 160 bytes a pair).
    // (A batch whose rows would not fit there either keeps the faster layout: 65 536 pairs
    // of about 350 letters 5.9 / 3.4 ms.)
    if (lay.bytes + 160ull * n > ALN_NOALLOC_WORKSPACE_BYTES) {
      std::vector<TaskDim> fine = td;
      make_tasks(16 * (tile ? tile : 16));
      Layout plain = lay_out(tile ? tile : 16, kWideOne);
      uint64_t least = 0; // boundary rows without those of short wide tasks
      for (const Item &it : plain.items)
        for (int32_t k = it.first; k < it.end; ++k)
          if (td[k].mmax > (it.wide >= 0 ? 64 : 16) * plain.R && (it.wide < 0 || it.wide == td[k].pa))
            least += align_up((uint64_t)(td[k].nmax + 1) * 8);
      if (least > ALN_NOALLOC_WORKSPACE_BYTES / 10 * 11) td.swap(fine);
      else lay = std::move(plain);
    }
    const int R = lay.R;
    pl->sw16_rows = R;
    pl->sw16_both = lay.form == kWideBoth;
    const int32_t HS = 16 * R, HB = 64 * R, HW = 128 * R; // strip heights: 16-lane group, wide
                                                          // item of two pairs, of one
    std::vector<Item> &items = lay.items;
    // longest item first: workgroups are dispatched in index order
    std::vector<uint64_t> steps(items.size());
    for (size_t k = 0; k < items.size(); ++k) steps[k] = (uint64_t)items[k].steps;
    pl->sw16_wide = 0;
    uint64_t bnd_bytes = 0;
    std::vector<uint64_t> bnd_rel;
    LaunchDesc L{};
    L.kind = K_SW16;
    L.rows = R;
    L.mode = ALN_LOCAL;
    L.first = 0;
    for (const int32_t at : order_desc(steps)) {
      const Item &it = items[(size_t)at];
      pl->sw16_items.push_back(
          alnk::Sw16Item{(int32_t)pl->sw16_tasks.size(), it.wide != -1 ? -1 : it.end - it.first});
      pl->sw16_wide += it.wide != -1;
      for (int32_t k = it.first; k < it.end; ++k) {
        const TaskDim &d = td[k];
        alnk::Sw16Task t;
        if (it.wide >= 0) {
          t.pa = it.wide;
          t.pb = -1;
          t.nstrips = nstr(pl->qlen[it.wide], HW);
          t.nmax = pl->rlen[it.wide];
        } else {
          t.pa = d.pa;
          t.pb = d.pb;
          t.nstrips = nstr(d.mmax, it.wide == kBoth ? HB : HS);
          t.nmax = d.nmax;
        }
        if (t.nmax == 0) t.nstrips = 0; // no column (nor one that a strip could leave to the next)
        t.bnd_off = 0;
        bnd_rel.push_back(t.nstrips > 1 ? bnd_bytes : ~0ULL);
        if (t.nstrips > 1) bnd_bytes += align_up((uint64_t)(t.nmax + 1) * (it.wide >= 0 ? 4 : 8), 16);
        pl->sw16_tasks.push_back(t);
        // the same pairs one by one (per-pair runs, always wide), sharing the
        // task's boundary row: a pair alone never has more strips, nor more
        // columns, than its task
        for (int h = 0; h < 2; ++h) {
          const int32_t pp = h ? t.pb : t.pa;
          if (pp < 0) continue;
          alnk::Sw16Task u;
          u.pa = pp;
          u.pb = -1;
          u.nstrips = pl->rlen[pp] > 0 ? nstr(pl->qlen[pp], HW) : 0;
          u.nmax = pl->rlen[pp];
          u.bnd_off = (int64_t)(pl->sw16_tasks.size() - 1); // task index, resolved below
          pl->sw16_single.push_back(u);
          pl->sw16_single_rows.push_back(R);
        }
      }
    }
    L.count = (int32_t)pl->sw16_tasks.size();
    pl->launches.push_back(L);
    // workspace: [sw16 tasks | items | single tasks | rerun counter | rerun queue |
    //             boundary rows]
    pl->sw16_off = 0;
    pl->sw16_items_off = align_up(sizeof(alnk::Sw16Task) * pl->sw16_tasks.size());
    pl->sw16_single_off =
        pl->sw16_items_off + align_up(sizeof(alnk::Sw16Item) * pl->sw16_items.size());
    pl->rerun_cnt_off = pl->sw16_single_off + align_up(sizeof(alnk::Sw16Task) * pl->sw16_single.size());
    pl->rerun_off = pl->rerun_cnt_off + kAlign;
    const uint64_t bnd_base = pl->rerun_off + align_up(sizeof(PairTask) * (size_t)n);
    for (size_t k = 0; k < pl->sw16_tasks.size(); ++k)
      pl->sw16_tasks[k].bnd_off = bnd_rel[k] == ~0ULL ? 0 : (int64_t)(bnd_base + bnd_rel[k]);
    for (alnk::Sw16Task &u : pl->sw16_single) u.bnd_off = pl->sw16_tasks[(size_t)u.bnd_off].bnd_off;
    pl->rerun.kind = K_RERUN;
    pl->rerun.rows = rerun_rows;
    pl->rerun.mode = ALN_LOCAL;
    pl->rerun.tb = false;
    pl->rerun.small = small;
    pl->rerun.first = 0;
    pl->rerun.count = n;
    pl->rerun.lds_bnd = rerun_bnd;
    pl->rerun.lds_prof = rerun_prof;
    for (int32_t i = 0; i < n; ++i) pl->cells += (int64_t)pl->qlen[i] * pl->rlen[i];
    pl->upload_bytes = pl->rerun_cnt_off;
    pl->tasks_bytes = bnd_base + bnd_bytes;
    pl->tb_base = pl->tasks_bytes;
    pl->tb_bytes = 0;
    pl->ws_bytes = pl->tasks_bytes;
    pl->cigar_words = 0;
    *plan = pl;
    return ALN_OK;
  }

  // ---- per-pair kernel choice: full-matrix strips, or the antidiagonal
  // kernel (band, X-drop) with a window of 64*RD diagonals
  struct Item {
    int32_t pair;
    int kind;
    int rows;
    double cost;
    int waves = 1; // full matrix / band strips: wavefronts per pair (strip pipeline);
                   // rolling blocks: lanes per pair
    int ring = 0;  // band strips: columns of the LDS boundary ring
    bool full = false; // rolling blocks: full matrix
  };
  // Launch order: by kernel and tile, each longest first, equal ones by pair.
  auto cls_of = [](const Item &it) {
    return ((it.kind * 128 + it.waves) * 64 + it.rows) * 2 + (it.full ? 1 : 0);
  };
  std::vector<int32_t> order; // of items
  // by class, the order inside each kept
  auto regroup = [&](const std::vector<Item> &v) {
    std::vector<std::pair<int32_t, int32_t>> classes; // and how many
    std::vector<int32_t> cls(v.size());
    for (size_t k = 0; k < v.size(); ++k) {
      cls[k] = cls_of(v[k]);
      size_t c = 0;
      while (c < classes.size() && classes[c].first != cls[k]) ++c;
      if (c == classes.size()) classes.push_back({cls[k], 0});
      ++classes[c].second;
    }
    if (classes.size() < 2) return;
    std::sort(classes.begin(), classes.end());
    int32_t sum = 0;
    for (auto &c : classes) {
      const int32_t here = c.second;
      c.second = sum;
      sum += here;
    }
    std::vector<int32_t> out(v.size());
    for (const int32_t k : order) {
      size_t c = 0;
      while (classes[c].first != cls[(size_t)k]) ++c;
      out[(size_t)classes[c].second++] = k;
    }
    order.swap(out);
  };
  auto sort_items = [&](const std::vector<Item> &v) {
    std::vector<uint64_t> cost(v.size()); // not negative, so its bits sort as it does
    for (size_t k = 0; k < v.size(); ++k) memcpy(&cost[k], &v[k].cost, sizeof cost[k]);
    order = order_desc(cost);
    regroup(v);
  };
  std::vector<Item> items;
  items.reserve(n);
  static const int kDiagRows[] = {2, 4, 8, 10, 16, 32};
  int srows = ctx->tuning.valid ? ctx->tuning.strip_rows : 0;
  if (ctx->force_strip_rows >= 0) srows = ctx->force_strip_rows;
  for (int32_t i = 0; i < n; ++i) {
    const int32_t M = pl->qlen[i], N = pl->rlen[i];
    if (M < 0 || N < 0) {
      delete pl;
      return fail(ctx, ALN_E_INVAL, "negative length at pair %d", i);
    }
    if ((int64_t)(M + (int64_t)N) * per_step >= (1LL << 29)) {
      delete pl;
      return fail(ctx, ALN_E_UNSUPPORTED, "pair %d too long for int32 scores", i);
    }
    Item it{i, K_STRIP, 0, 0.0};
    const bool band_is_full = p.prune == ALN_BAND && (M == 0 || p.band_w >= std::max(M, N));
    if (p.prune == ALN_FULL || band_is_full) {
      it.rows = srows ? srows : choose_strip_rows(M, N);
      it.cost = (double)M * N;
      pl->cells += (int64_t)M * N;
    } else {
      it.kind = K_DIAG;
      if (p.mode != ALN_GLOBAL && (int64_t)std::max(hs.max_s, 1) * std::min(M, N) >= (1 << 20)) {
        delete pl;
        return fail(ctx, ALN_E_UNSUPPORTED, "pair %d: best score may exceed 2^20", i);
      }
      if (p.prune == ALN_BAND) {
        const int64_t w = p.band_w;
        // strips (band_kernel 2..5: one or four wavefronts per pair, 4 or 2
        // rows per lane): a strip's columns and 10 spare ones fit one LDS ring
        // of at most 2048, and the pipeline's stamps s*(N+1) + column fit 31
        // bits
        int bk = ctx->force_band_kernel
                     ? ctx->force_band_kernel
                     : (ctx->tuning.valid ? ctx->tuning.band_kernel : 0);
        if (bk == 0) bk = 2 * w + 1 >= 256 ? 5 : 1; // wide bands: strips, four wavefronts of 2 rows
        const int brows = (bk == 4 || bk == 5) ? 2 : 4;
        const int64_t cols = M > 0 && N > 0 ? alnk::band_strip_cols(M, N, (int32_t)std::min<int64_t>(w, 1 << 28), brows) : 0;
        const int64_t ring = std::max<int64_t>(64, (cols + 10 + 15) / 16 * 16);
        const int64_t nsb = (M + 64LL * brows - 1) / (64LL * brows);
        const bool strip_fit = M > 0 && N > 0 && ring <= 2048 && w < (1 << 28) &&
                               nsb * ((int64_t)N + 1) + N < (1LL << 31);
        if (bk >= 2 && strip_fit) {
          it.kind = K_BAND;
          it.rows = brows;
          it.waves = (bk == 3 || bk == 5) ? alnk::kStripPipeWaves : 1;
          it.ring = (int)ring;
          it.cost = (double)nsb * (double)(cols + 63) * brows;
        } else {
          int64_t width = 2 * w + 6 + ((2 * w + 2) * std::abs((int64_t)N - M) + M - 1) / std::max(M, 1);
          width = std::min<int64_t>(width, 2LL * std::min(M, N) + 6);
          it.rows = 0;
          for (int r : kDiagRows)
            if (64LL * r - 6 >= width && (!p.want_cigar || r <= 16)) { it.rows = r; break; }
          if (it.rows == 0) {
            delete pl;
            return fail(ctx, ALN_E_UNSUPPORTED, "pair %d: band of %lld diagonals exceeds the window",
                        i, (long long)width);
          }
          it.cost = (double)(M + N) * it.rows;
        }
        pl->cells += band_cells(M, N, p.band_w);
      } else {
        it.rows = ctx->tuning.valid ? ctx->tuning.xdrop_rows : 4;
        if (ctx->force_xdrop_rows) it.rows = ctx->force_xdrop_rows;
        it.cost = (double)(M + N);
      }
    }
    items.push_back(it);
  }
  // Strip pipeline: when the full-matrix pairs are too few to give every
  // SIMD a wavefront of its own, a pair of several strips runs on the
  // wavefronts of one workgroup, its strips handed down through LDS -- unless
  // a fixed strip height is tuned or forced.  By default, with at most three
  // quarters of a wavefront per SIMD, four wavefronts of 4 rows per lane
  // (256-row strips).  Tuned tiles ask for it (4) or for eight wavefronts of
  // 2 rows (2; 128-row strips, two wavefronts per SIMD of the CU: measured
  // 3% slower on 1 kbp pairs, where each strip's start behind the one above
  // sets the pace).  Boundary buffers hold whole rows, which bounds N.
  //
  // In the automatic choice the pipelined pairs run on the band strips with a
  // band past the matrix (the same four-wavefront schedule, 256-row strips):
  // that kernel's rotating lane-0 feeds and eight-step code stores take
  // about 18% less time on 1 kbp pairs.  Its LDS ring holds a strip's
  // columns and 10 more, so N <= 2038.
  pl->strip_band_w = p.prune == ALN_BAND ? std::min(p.band_w, 1 << 28) : (1 << 28); // (columns are added to it)
  if (srows == 0 || srows == 2 || srows == 4) {
    int64_t n_full = 0;
    for (const Item &it : items) n_full += it.kind == K_STRIP;
    const int64_t simds = 4LL * ctx->cus;
    int R = 0, G = 0;
    if (srows == 2) {
      R = 2;
      G = alnk::kStripPipeWaves2;
    } else if (srows == 4 || n_full * 4 <= simds * 3) {
      R = 4;
      G = alnk::kStripPipeWaves;
    }
    for (Item &it : items) {
      if (it.kind != K_STRIP || G == 0) continue;
      const int32_t M = pl->qlen[it.pair], N = pl->rlen[it.pair];
      const uint64_t bnd = align_up((uint64_t)(N + 1) * 8, 16);
      const uint64_t prof = small ? 0 : align_up((uint64_t)hs.alphabet * 64 * R, 16);
      if ((srows == 0 || srows == 2) && M > 64 * R && N <= 2038 &&
          pl->strip_band_w >= std::max(M, N)) {
        const int64_t ring = std::max<int64_t>(64, ((int64_t)N + 10 + 15) / 16 * 16);
        it.kind = K_BAND;
        it.rows = R;
        it.waves = G;
        it.ring = (int)ring;
        it.cost = (double)((M + 64LL * R - 1) / (64LL * R)) * (double)(N + 63) * R;
      } else if (M > 64 * R && alnk::strip_lds_bytes(G, (int)bnd, (int)prof, N) <= 160 * 1024) {
        it.rows = R;
        it.waves = G;
      } else if (srows != 0) {
        it.rows = choose_strip_rows(M, N); // a one-strip pair, or one too wide for the LDS
      }
    }
  }
  // The choice so far decides which batches are refused (strips whose rows or
  // profiles outgrow LDS) and the order of the CIGAR slots, whichever kernel
  // below takes a pair over: both stay what they were.
  {
    struct Group {
      int32_t rows, waves, n;
      bool multi;
    };
    std::vector<Group> groups;
    for (const Item &it : items) {
      if (it.kind != K_STRIP) continue;
      size_t g = 0;
      while (g < groups.size() && (groups[g].rows != it.rows || groups[g].waves != it.waves)) ++g;
      if (g == groups.size()) groups.push_back(Group{it.rows, it.waves, 0, false});
      groups[g].n = std::max(groups[g].n, pl->rlen[it.pair]);
      groups[g].multi = groups[g].multi || pl->qlen[it.pair] > 64 * it.rows;
    }
    for (const Group &g : groups) {
      const int bnd = g.multi ? (int)align_up((uint64_t)(g.n + 1) * 8, 16) : 0;
      const int prof = small ? 0 : (int)align_up((uint64_t)hs.alphabet * 64 * g.rows, 16);
      if (alnk::strip_lds_bytes(g.waves, bnd, prof, g.n) > 160 * 1024) {
        delete pl;
        return fail(ctx, ALN_E_UNSUPPORTED,
                    "full-matrix pairs with N = %d and M > %d need more LDS than a CU has", g.n,
                    64 * g.rows);
      }
    }
  }
  sort_items(items);
  const bool codes = p.want_cigar && !dyn_prune; // the tasks' own (not X-drop's, below)
  std::vector<int64_t> slot;
  uint64_t cg_off = 0;
  if (codes) {
    slot.resize(n);
    for (int32_t k : order) {
      const Item &it = items[(size_t)k];
      slot[it.pair] = (int64_t)cg_off;
      cg_off += (uint64_t)pl->qlen[it.pair] + pl->rlen[it.pair] + 1;
    }
  }
  // bytes of a pair's traceback codes where an item runs it
  auto code_bytes = [&](const Item &it) -> uint64_t {
    const int32_t M = pl->qlen[it.pair], N = pl->rlen[it.pair];
    const uint64_t strips = (uint64_t)((M + 64LL * it.rows - 1) / (64LL * it.rows));
    if (it.kind == K_STRIP) return strips * (uint64_t)(N + 63) * 64 * (uint64_t)(it.rows / 2);
    if (it.kind == K_BAND)
      return strips * 64 * (uint64_t)alnk::band_code_steps(M, N, pl->strip_band_w, it.rows) *
             (uint64_t)(it.rows / 2);
    if (it.kind == K_ROLL)
      return (uint64_t)((M + it.rows - 1) / it.rows) *
             (uint64_t)alnk::roll_code_steps(M, N, it.full ? 1 << 28 : p.band_w, it.rows) *
             (uint64_t)(it.rows / 2);
    const uint64_t nk = (uint64_t)M + N + 1;
    return (nk + 63) / 64 * 64 * 4 + ((uint64_t)(M + N) / 2 + 1) * 64 * 8;
  };
  std::vector<Item> own; // the choice so far, where a pair is moved and there are codes
  bool moved = false;    // some pair runs elsewhere
  auto move_away = [&] {
    if (!moved && codes) own = items;
    moved = true;
  };
  // Narrow bands: rolling blocks where a shape fits, else the band strips.
  // (a tuned or forced choice of the antidiagonal kernel: rolling blocks only)
  const int band_asked = ctx->force_band_kernel ? ctx->force_band_kernel
                                                : (ctx->tuning.valid ? ctx->tuning.band_kernel : 0);
  if (p.prune == ALN_BAND && band_asked <= 1 && n >= kStripBandPairs) {
    auto strips = [&](Item &it, int32_t least) {
      const int32_t M = pl->qlen[it.pair], N = pl->rlen[it.pair];
      if (it.kind != K_DIAG || M < least || N < 1) return;
      const int64_t ring = (alnk::band_strip_cols(M, N, p.band_w, 2) + 10 + 15) / 16 * 16;
      if (ring > 2048 || ((M + 127LL) / 128) * ((int64_t)N + 1) + N >= (1LL << 31)) return;
      move_away();
      it.kind = K_BAND;
      it.rows = 2;
      it.waves = alnk::kStripPipeWaves;
      it.ring = (int)std::max<int64_t>(64, ring);
    };
    bool beside = false; // some pairs run on strips
    for (Item &it : items) {
      if (it.kind != K_DIAG) continue;
      const int32_t M = pl->qlen[it.pair], N = pl->rlen[it.pair];
      if (M < 1 || N < 1) continue;
      int rows = 0, lanes = 0;
      if (small && n >= kRollPairs) roll_shape(ctx, n, M, N, p.band_w, &rows, &lanes);
      if (rows) {
        move_away();
        it.kind = K_ROLL;
        it.rows = rows;
        it.waves = lanes;
      } else if (band_asked == 0 && p.band_w < 128) {
        strips(it, 128);
        beside = beside || it.kind == K_BAND;
      }
    }
    // Shorter pairs beside them take strips too, rather than a launch of the antidiagonal kernel
    // after theirs: 16 pairs of 100..150 rows, 20 letters, paths, 91 us; in two launches 270, all on
    // antidiagonals 222.  (Pairs of 15..25 rows take less there from two a SIMD on: 2 100 63
    // against 55 us, 30 000 468 against 316; of 30..60 30 000 531 against 648.)
    if (beside)
      for (Item &it : items) strips(it, n <= 4LL * ctx->cus ? 1 : 32);
  }
  // Full matrix, no strip height tuned or forced.
  //
  // Up to a quarter of a pair per SIMD, where a launch takes its longest
  // pair's time, all pairs run on the band strips, so that the batch is one
  // launch and one walk: with 2 rows per lane (128-row strips) while no pair
  // has more than four of them.  16 pairs of 60..300 bp with paths: 124 us
  // against 277 with the one-strip pairs in a launch of their own.
  //
  // Short pairs of larger batches run as rolling blocks, four to a wavefront
  // of 16 lanes each, where a strip of 64 lanes would be a third full: 8 192
  // reads of 150 bp against 150..320 bp windows, LOCAL with paths, 0.30 ms
  // against 0.88.  Up to 160 rows a pair takes no longer there than on its own
  // wavefront, of 161..256 rows (16 a lane) twice as long, so those only past
  // two pairs a SIMD (LOCAL with paths against longer references three: 2 100 pairs of
  // 30..250 rows against 60..500 415 us on strips, 523 rolling).  One launch,
  // its rows a lane by the longest query, until eight pairs a SIMD; from there on by each
  // pair's, and beside longer pairs, but for rows a lane that few pairs take: beside the
  // strips that is one more launch of a pair's time (9 000 pairs, half of 20..60 rows, half
  // of 250..600, some hundred of them up to 256, LOCAL with paths: 1.99 ms all on strips, 2.15
  // with such a launch, 1.96 without).
  if (srows == 0) {
    int64_t n_full = 0;
    int32_t fullM = 0, fullN = 0;
    auto whole = [&](const Item &it) {
      return it.kind == K_STRIP ||
             (it.kind == K_BAND && pl->strip_band_w >= std::max(pl->qlen[it.pair], pl->rlen[it.pair]));
    };
    for (const Item &it : items)
      if (whole(it)) {
        ++n_full;
        fullM = std::max(fullM, pl->qlen[it.pair]);
        fullN = std::max(fullN, pl->rlen[it.pair]);
      }
    const int64_t simds = 4LL * ctx->cus;
    const bool few = n >= kStripBandPairs && n_full * 4 <= simds && fullN <= 2038;
    const bool few8 =
        alnk::band_lds_bytes(alnk::kStripPipeWaves2, (fullN + 10 + 15) / 16 * 16,
                             small ? 0 : (int)align_up((uint64_t)hs.alphabet * 64 * 4, 16)) <= 160 * 1024;
    const bool split = n_full > 8 * simds;
    const int64_t from16 = (p.mode == ALN_LOCAL && p.want_cigar && 10LL * fullN > 13LL * fullM ? 3 : 2) * simds;
    auto roll_rows = [](int32_t top) { return top <= 128 ? 8 : (top <= 160 ? 10 : 16); };
    auto rolls = [&](const Item &it) {
      const int32_t M = pl->qlen[it.pair], N = pl->rlen[it.pair];
      return it.kind == K_STRIP && small && n_full >= kRollPairs && N < 65536 && M <= 256 && M >= 1 && N >= 1 &&
             (split || fullM <= 160 || (fullM <= 256 && n_full > from16));
    };
    int64_t rolling = 0, by_rows[17] = {};
    if (split && !few)
      for (const Item &it : items)
        if (whole(it) && rolls(it)) {
          ++rolling;
          ++by_rows[roll_rows(pl->qlen[it.pair])];
        }
    const bool beside = split && rolling < n_full;
    for (Item &it : items) {
      const int32_t M = pl->qlen[it.pair], N = pl->rlen[it.pair];
      if (!whole(it) || M < 1 || N < 1) continue;
      if (few) {
        move_away();
        it.kind = K_BAND;
        // as many strips at a time as there are, of the rows that run shortest: two or
        // four rows a lane on four / eight wavefronts, M = N, fill us:
        //   500: 139, 144 / 140, 145   600: 196, 182 / 172, 182   800: 289, 239 / 246, 238
        //   1 000: 365, 277 / 302, 277   1 300: 633, 582 / 438, 507
        //   1 600: 972, 718 / 682, 626   2 000: 1 484, 883 / 923, 779
        it.rows = fullM <= 640 || (fullM > 1024 && fullM <= 1408) ? 2 : 4;
        it.waves = fullM <= 512 || (fullM > 640 && fullM <= 1024) ? alnk::kStripPipeWaves
                                                                  : alnk::kStripPipeWaves2;
        if (!few8) { // eight wavefronts' rings and profiles do not fit
          it.rows = fullM <= 512 ? 2 : 4;
          it.waves = alnk::kStripPipeWaves;
        }
        it.ring = (int)std::max<int64_t>(64, ((int64_t)N + 10 + 15) / 16 * 16);
      } else if (rolls(it)) {
        const int rows = roll_rows(split ? M : fullM);
        if (beside && by_rows[rows] * 2 < simds) continue;
        move_away();
        it.kind = K_ROLL;
        it.full = true;
        it.rows = rows;
        it.waves = 16;
      }
    }
  }
  // X-drop without traceback under match / mismatch scoring on a small
  // alphabet runs on the lanes kernel (4 to 16 sides per wavefront) when its
  // arithmetic fits: offset-frame scores in one byte, the out-of-range
  // penalty (-128) below every threshold (X < 128 + 2|e|), end cells in 16
  // bits and keys (score << 6, or 7) in 31.  Z-drop too, scores only (its form
  // masks removed and out-of-range cells itself, so Z has no bound).
  const bool zd = p.prune == ALN_ZDROP;
  const bool lanes_fit =
      (p.prune == ALN_XDROP || zd) && hs.match_mismatch && hs.alphabet <= 4 &&
      (zd || (int64_t)p.xdrop <= 127 - 2LL * hs.gap_extend) && hs.match - 2 * hs.gap_extend <= 127 &&
      hs.mismatch - 2 * hs.gap_extend >= -128 && maxM <= 65535 && maxN <= 65535 &&
      ((int64_t)maxM + maxN) * (1 - hs.gap_extend + std::max(hs.match, 0)) < (1LL << 23);
  const bool lanes_ok = lanes_fit && !p.want_cigar;
  // The other families' codes take up to three times the bytes of a pair's own (512 x 60
  // full matrix, two rows a lane instead of eight: 2.2): not past what a call without
  // allocation has where its own would fit.  (The workspace is the task list and the
  // codes.)
  std::vector<uint64_t> bytes; // of each item's codes
  if (codes) {
    auto workspace = [&](const std::vector<Item> &v) {
      uint64_t sum = align_up(sizeof(PairTask) * (size_t)std::max(n, 1));
      bytes.resize(v.size());
      for (size_t k = 0; k < v.size(); ++k) sum += bytes[k] = align_up(code_bytes(v[k]));
      return sum;
    };
    constexpr uint64_t lim = ALN_NOALLOC_WORKSPACE_BYTES;
    const uint64_t now = workspace(items);
    if (moved && now > lim && now <= 4 * lim && (uint64_t)pl->cells / 2 <= lim) { // 4 bits a cell at least
      std::vector<uint64_t> elsewhere;
      elsewhere.swap(bytes);
      if (workspace(own) <= lim) {
        items.swap(own);
        moved = false;
      } else {
        bytes.swap(elsewhere);
      }
    }
  }
  if (moved) regroup(items); // longest first by the first choice's cost
  uint64_t tb_off = 0;
  auto at = [&](size_t k) -> const Item & { return items[(size_t)order[k]]; };
  for (size_t k = 0; k < items.size();) {
    size_t e = k;
    int32_t grpN = 0, grpRing = 0;
    bool multi = false;
    while (e < items.size() && at(e).kind == at(k).kind && at(e).rows == at(k).rows &&
           at(e).waves == at(k).waves && at(e).full == at(k).full) {
      grpN = std::max(grpN, pl->rlen[at(e).pair]);
      grpRing = std::max(grpRing, at(e).ring);
      if (at(e).kind == K_STRIP && pl->qlen[at(e).pair] > 64 * at(e).rows) multi = true;
      ++e;
    }
    LaunchDesc L{};
    L.kind = at(k).kind;
    L.rows = at(k).rows;
    L.mode = p.mode;
    if (L.kind == K_DIAG && dyn_prune) {
      // Z-drop by default takes the 128-cell window in large batches, which holds
      // what the one-side kernel's first window holds, unless Z lets regions reach
      // so far that nearly every side outgrows that (at e = -1, 17 000 sides of 150..1 500
      // bp at Z = 15 / 30 / 60 / 100, ms with lanes 23.0 / 21.4 / 24.6 / 24.6, one side a
      // wavefront 21.6 / 19.0 / 21.9 / 22.3).  Tuned to the
      // lanes form it takes the 64-cell window where regions fit that (at Z =
      // 100, e = -2 nearly every side outgrows 64: 100 000 sides 111.5 ms there, 48.2 on
      // 128; at Z = 40 22.6 and 40.1).
      const bool lanes_asked =
          (ctx->force_xdrop_sides ? ctx->force_xdrop_sides : (ctx->tuning.valid ? ctx->tuning.xdrop_sides : 0)) == 16;
      const bool narrow = zdrop_within(hs, p, 60);
      const bool zd_wide =
          zd && lanes_ok &&
          (lanes_asked ? !narrow
                       : (!ctx->tuning.valid && !ctx->force_xdrop_sides &&
                          (int64_t)(e - k) >= zdrop_lanes_from(ctx) && zdrop_within(hs, p, kZdropReach)));
      L.sides = ctx->tuning.valid ? ctx->tuning.xdrop_sides : ((lanes_ok && (!zd || zd_wide)) ? 16 : 1);
      if (ctx->force_xdrop_sides) L.sides = ctx->force_xdrop_sides;
      if (L.sides == 16 && !lanes_ok) L.sides = 1;
      if (L.sides == 4 && L.rows != 8) L.sides = 1;
      if (L.sides == 16) {
        L.lps = zd ? (zd_wide ? 8 : 4) : lanes_per_side(ctx, (int64_t)(e - k));
        L.window = zd_wide ? 128 : 64;
        const int per = 64 / L.lps;
        const int64_t want = ((int64_t)(e - k) + per - 1) / per;
        const int64_t fit = (int64_t)ctx->cus * alnk::xdrop_lanes_waves(false, zd, L.lps);
        L.grid = (int)std::max<int64_t>(1, std::min(want, fit));
      }
    }
    L.tb = p.want_cigar != 0 && !dyn_prune; // X-drop codes come from a second pass
    L.small = small;
    L.first = (int32_t)pl->tasks.size();
    L.count = (int32_t)(e - k);
    L.waves = at(k).waves;
    L.full = at(k).full;
    if (L.kind == K_BAND) {
      L.lds_bnd = grpRing * 8;
      L.lds_prof = small ? 0 : (int32_t)align_up((uint64_t)hs.alphabet * 64 * L.rows, 16);
      L.max_n = grpN;
    }
    if (L.kind == K_STRIP) {
      L.lds_bnd = multi ? (int32_t)align_up((uint64_t)(grpN + 1) * 8, 16) : 0;
      L.lds_prof = small ? 0 : (int32_t)align_up((uint64_t)hs.alphabet * 64 * L.rows, 16);
      L.max_n = grpN;
    }
    for (size_t q = k; q < e; ++q) {
      const int32_t i = at(q).pair;
      const int32_t M = pl->qlen[i], N = pl->rlen[i];
      PairTask t;
      memset(&t, 0, sizeof t);
      t.pair = i;
      t.rows = L.rows;
      t.tb_off = -1;
      if (codes) {
        t.tb_off = (int64_t)tb_off;
        tb_off += bytes[(size_t)order[q]];
        t.cigar_off = slot[i];
        t.cigar_cap = M + N + 1;
      }
      pl->tasks.push_back(t);
    }
    pl->launches.push_back(L);
    k = e;
  }
  // X-drop / Z-drop with CIGAR: a second task list, one task per pair with
  // 4 diagonals per lane, for the traceback pass and the walk.  Codes take 2
  // bytes per lane and antidiagonal pair, plus the window base per
  // antidiagonal; the pass stops at the end cell's antidiagonal.
  if (dyn_prune && p.want_cigar) {
    pl->xtb_first = (int32_t)pl->tasks.size();
    pl->xtb_count = n;
    // the lanes kernel writes the codes where its arithmetic fits,
    // unless a tuned tile other than its own asks for the one-side pass
    const int tuned_sides = ctx->force_xdrop_sides
                                ? ctx->force_xdrop_sides
                                : (ctx->tuning.valid ? ctx->tuning.xdrop_sides : 16);
    pl->xtb_lanes = lanes_fit && !zd && tuned_sides == 16;
    if (pl->xtb_lanes) {
      pl->xtb_lps = lanes_per_side(ctx, n);
      const int per = 64 / pl->xtb_lps;
      const int64_t want = ((int64_t)n + per - 1) / per;
      const int64_t fit = (int64_t)ctx->cus * alnk::xdrop_lanes_waves(true, false, pl->xtb_lps);
      pl->xtb_grid = (int)std::max<int64_t>(1, std::min(want, fit));
    }
    std::vector<uint64_t> len(n);
    for (int32_t i = 0; i < n; ++i) len[i] = (uint64_t)pl->qlen[i] + (uint64_t)pl->rlen[i];
    for (const int32_t i : order_desc(len)) {
      const int32_t M = pl->qlen[i], N = pl->rlen[i];
      PairTask t;
      memset(&t, 0, sizeof t);
      t.pair = i;
      t.rows = 4;
      const uint64_t nk = (uint64_t)M + N + 1;
      const uint64_t bytes = (nk + 63) / 64 * 64 * 4 + ((uint64_t)(M + N) / 2 + 1) * 64 * 2;
      t.tb_off = (int64_t)tb_off;
      tb_off += align_up(bytes);
      t.cigar_off = (int64_t)cg_off;
      t.cigar_cap = M + N + 1;
      cg_off += (uint64_t)(M + N + 1);
      pl->tasks.push_back(t);
    }
    pl->first_diag_tb = pl->xtb_first;
    pl->n_diag_tb = n;
  }
  // walk ranges: strip tasks come first (kind order), then antidiagonal tasks
  if (p.want_cigar && !dyn_prune) {
    for (const LaunchDesc &L : pl->launches) {
      if (L.kind == K_STRIP) pl->n_strip_tb += L.count;
      if (L.kind == K_DIAG) {
        if (pl->n_diag_tb == 0) pl->first_diag_tb = L.first;
        pl->n_diag_tb += L.count;
      }
      if (L.kind == K_BAND) {
        if (pl->n_band_tb == 0) pl->first_band_tb = L.first;
        pl->n_band_tb += L.count;
      }
      if (L.kind == K_ROLL) {
        pl->roll_full_tb = pl->roll_full_tb || L.full;
        if (pl->n_roll_tb == 0) pl->first_roll_tb = L.first;
        pl->n_roll_tb += L.count;
      }
    }
  }
  pl->xdrop = dyn_prune; // X-drop or Z-drop: widening queues
  pl->tasks_bytes = align_up(sizeof(PairTask) * std::max<size_t>(pl->tasks.size(), 1));
  pl->upload_bytes = sizeof(PairTask) * pl->tasks.size();
  if (pl->xdrop) {
    pl->widen_cnt_off = pl->tasks_bytes;
    pl->widen_off[0] = pl->widen_cnt_off + kAlign;
    pl->widen_off[1] = pl->widen_off[0] + align_up(sizeof(PairTask) * (size_t)std::max(n, 1));
    pl->widen_off[2] = pl->widen_off[1] + align_up(sizeof(PairTask) * (size_t)std::max(n, 1));
    pl->tasks_bytes = pl->widen_off[2] + (pl->xtb_lanes ? align_up(sizeof(PairTask) * (size_t)std::max(n, 1)) : 0);
  }
  pl->tb_base = pl->tasks_bytes;
  pl->tb_bytes = tb_off;
  pl->ws_bytes = pl->tb_base + pl->tb_bytes;
  pl->cigar_words = cg_off;
  *plan = pl;
  return ALN_OK;
}

void alnrt::plan_stage(const aln_plan *pl, void *dst) {
  uint8_t *d = static_cast<uint8_t *>(dst);
  if (pl->fold) {
    memcpy(d, pl->fold_tasks.data(), sizeof(alnk::FoldTask) * pl->fold_tasks.size());
    return;
  }
  if (!pl->sw16_tasks.empty()) {
    memcpy(d + pl->sw16_off, pl->sw16_tasks.data(), sizeof(alnk::Sw16Task) * pl->sw16_tasks.size());
    memcpy(d + pl->sw16_items_off, pl->sw16_items.data(),
           sizeof(alnk::Sw16Item) * pl->sw16_items.size());
    memcpy(d + pl->sw16_single_off, pl->sw16_single.data(),
           sizeof(alnk::Sw16Task) * pl->sw16_single.size());
  } else if (!pl->tasks.empty()) {
    memcpy(d, pl->tasks.data(), sizeof(PairTask) * pl->tasks.size());
  }
}

extern "C" {

aln_status aln_plan_create(aln_ctx *ctx, int32_t scoring_id, const aln_params *params, int32_t n,
                           const int32_t *q_len_host, const int32_t *r_len_host, aln_plan **plan,
                           aln_footprint *fp) {
  aln_plan *pl = nullptr;
  aln_status st = plan_build(ctx, scoring_id, params, n, q_len_host, r_len_host, &pl);
  if (st != ALN_OK) return st;
  if (alnrt::plan_alloc_staging(pl) != ALN_OK) {
    delete pl;
    return fail(ctx, ALN_E_NOMEM, "staging for %llu bytes", (unsigned long long)pl->upload_bytes);
  }
  plan_stage(pl, pl->pinned);
  if (fp) {
    fp->workspace_bytes = pl->ws_bytes;
    fp->traceback_bytes = pl->tb_bytes;
    fp->cigar_words = pl->cigar_words;
    fp->cells = pl->cells;
  }
  *plan = pl;
  return ALN_OK;
}

void aln_plan_destroy(aln_plan *plan) {
  if (!plan) return;
  if (plan->gexec) (void)hipGraphExecDestroy(plan->gexec);
  if (plan->graph) (void)hipGraphDestroy(plan->graph);
  if (plan->pinned && plan->own_pinned) {
    if (plan->host_staging) std::free(plan->pinned);
    else (void)hipHostFree(plan->pinned);
  }
  delete plan;
}

} // extern "C"

aln_status alnrt::exec_check(aln_ctx *ctx, aln_plan *plan, const aln_batch *b, void *d_ws,
                             uint64_t ws_bytes, aln_result *d_res, uint32_t *d_cigar,
                             uint64_t cigar_words) {
  if (!ctx || !plan || !b || plan->ctx != ctx) return fail(ctx, ALN_E_INVAL, "bad context or plan");
  if (plan->fold) return fail(ctx, ALN_E_INVAL, "a folding plan runs with aln_fold_execute");
  if (b->n != plan->n) return fail(ctx, ALN_E_INVAL, "batch has %d pairs, plan %d", b->n, plan->n);
  if (plan->n == 0) return ALN_OK;
  if (!d_res || !b->q_off || !b->q_len || !b->r_off || !b->r_len)
    return fail(ctx, ALN_E_INVAL, "null device pointer");
  if (!d_ws || ws_bytes < plan->ws_bytes)
    return fail(ctx, ALN_E_CAPACITY, "workspace %llu < %llu bytes", (unsigned long long)ws_bytes,
                (unsigned long long)plan->ws_bytes);
  if (plan->p.want_cigar && (!d_cigar || cigar_words < plan->cigar_words))
    return fail(ctx, ALN_E_CAPACITY, "CIGAR buffer %llu < %llu words",
                (unsigned long long)cigar_words, (unsigned long long)plan->cigar_words);
  if (ctx->device < 0) return fail(ctx, ALN_E_DEVICE, "the context has no device");
  return ALN_OK;
}

aln_status alnrt::plan_alloc_staging(aln_plan *pl) {
  const size_t bytes = (size_t)std::max<uint64_t>(pl->upload_bytes, 1);
  if (pl->ctx->device < 0) {
    pl->pinned = std::malloc(bytes);
    pl->host_staging = true;
    return pl->pinned ? ALN_OK : ALN_E_NOMEM;
  }
  return hipHostMalloc(&pl->pinned, bytes, hipHostMallocDefault) == hipSuccess ? ALN_OK
                                                                               : ALN_E_NOMEM;
}

extern "C" {

// Wavefronts a pair for the walks of n pairs of up to rows rows (band
// layouts).  A walk is a serial chain, so more wavefronts shorten the launch until
// they no longer fit the chip at once (16 a CU); each share costs up to half its
// rows again for its guess.  Measured, 16 / 8 / 4 / 1 wavefronts in ms: 384
// pairs of 10..100 kbp 4.2 / 5.6 / 9.6 / 15.9; 1 000 of them 8.9 / 9.1 / 9.9 /
// 16.7; 2 048 of 1..9 kbp 1.14 / 0.82 / 0.70 / 1.20; 256 of 1 kbp 0.073 / 0.078 /
// 0.099 / 0.147; 700 of 0.5 kbp 0.138 / 0.103 / 0.083 / 0.103.
static int walk_shares(const aln_ctx *ctx, int64_t n, int32_t rows) {
  const int64_t simds = 4LL * ctx->cus;
  const int by_n = n * 2 <= simds ? 16 : (n <= simds ? 8 : (n <= 4 * simds ? 4 : 1));
  const int by_rows = rows >= 128 * 16 ? 16 : (rows >= 128 * 7 ? 8 : (rows >= 128 * 4 ? 4 : 1));
  return std::min(by_n, by_rows);
}

static aln_status run_plan(aln_ctx *ctx, aln_plan *plan, const aln_batch *b, void *d_ws,
                           aln_result *d_res, uint32_t *d_cigar, hipStream_t st, bool per_pair) {
  if (plan->n == 0) return ALN_OK;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  uint8_t *ws = static_cast<uint8_t *>(d_ws);
  PairTask *dtasks = reinterpret_cast<PairTask *>(ws);
  if (plan->upload_bytes)
    HIP_TRY(ctx, hipMemcpyAsync(ws, plan->pinned, plan->upload_bytes, hipMemcpyHostToDevice, st));
  alnk::BatchPtrs bp{b->q, b->q_off, b->q_len, b->r, b->r_off, b->r_len};
  const DevScoring *dsc = ctx->dsc[plan->scoring_id];
  const DevScoring &hsc = ctx->hsc[plan->scoring_id];
  const bool sw16 = !plan->sw16_tasks.empty();
  int32_t *rerun_cnt = sw16 ? reinterpret_cast<int32_t *>(ws + plan->rerun_cnt_off) : nullptr;
  PairTask *rerun_q = sw16 ? reinterpret_cast<PairTask *>(ws + plan->rerun_off) : nullptr;

  int32_t *widen_cnt = plan->xdrop ? reinterpret_cast<int32_t *>(ws + plan->widen_cnt_off) : nullptr;
  // counters: sw16 re-run queue; X-drop widening queues (2), the lanes
  // kernel's work queue (2) and its queue of pairs for the one-side pass with
  // codes, or Z-drop's third widening queue (1)
  alnk::ValidateArgs va{bp, plan->n, hsc.alphabet, d_res, sw16 ? rerun_cnt : widen_cnt,
                        sw16 ? 1 : (plan->xdrop ? 5 : 0)};
  HIP_TRY(ctx, timed_launch(ctx, "validate", st, [&] { return alnk::launch_validate(va, st); }));

  if (!plan->launches.empty() && plan->launches[0].kind == K_SEARCH) {
    const LaunchDesc &L = plan->launches[0];
    alnk::SearchArgs sa{bp,      dtasks,  L.count, d_res,    L.lds_bnd, L.lds_prof, L.lds_f,
                        L.waves, L.pen_x, L.pen_o, L.pen_e, L.ring_h,  L.ring_e,  L.pen_g, 0, 0,
                        L.waves == 1, hsc.alphabet <= 4};
    if (sa.two_bit) { // (the plan's sizes are those of bytes)
      sa.lds_q = (int32_t)align_up((uint64_t)plan->max_m / 4 + 8, 16);
      sa.lds_r = (int32_t)align_up((uint64_t)plan->max_n / 4 + 8, 16);
    }
    // with a diagonal cap: a capped pass, then full rows for the pairs it marked
    std::pair<const char *, alnk::SearchArgs> passes[2];
    int npass = 0;
    if (L.dcap > 0) {
      alnk::SearchArgs c = sa;
      c.lds_f = L.lds_fc;
      c.dcap = L.dcap;
      passes[npass++] = {L.pen_x > 0 ? "search_affine" : "search", c};
      sa.pass = 1;
      passes[npass++] = {L.pen_x > 0 ? "search_affine_wide" : "search_wide", sa};
    } else {
      passes[npass++] = {L.pen_x > 0 ? "search_affine" : "search", sa};
    }
    for (int ip = 0; ip < npass; ++ip) {
      alnk::SearchArgs &x = passes[ip].second;
      // Wavefronts a pair, by how many pairs a CU holds at a time: a score's diagonals
      // are few, and what a wavefront spends on a score whatever it has to do
      // counts where many pairs share the CU; where few do, they wait for a
      // score's chain.  1 / 2 / 4 / 8 wavefronts, us, edit distance: 30 000 pairs of
      // 100..200 nt (32 and more a CU) 49 / 73 / 126 / 234, 4 096 of 2 000 (eight)
      // 187 / 161 / 169 / 273, 1 000 of 7..8 knt (two) 1 240 / 808 / 565 / 464;
      // gap-affine, 4 096 of 2 000 (seven) 1 684 / 1 142 / 1 047 / 1 485, 64 of
      // 2 000 628 / 398 / 276 / 221.  (Capped rows are those of long pairs, with wide
      // scores: 4 096 of 2 000 nt, sixteen a CU, 140 / 134 us, at 20% 917 / 762.)
      if (!x.one_row) {
        const int64_t rows = x.pen_x > 0 ? x.ring_h + 2 * x.ring_e : 2;
        const int64_t lds = (int64_t)x.lds_q + x.lds_r + rows * x.lds_f;
        const int64_t held = std::min<int64_t>(ctx->lds_per_cu / lds,
                                               per_pair ? 1 : ((int64_t)L.count + ctx->cus - 1) / ctx->cus);
        x.waves = held >= (x.pen_x == 0 && x.dcap > 0 ? 24 : 16) ? 1 : held >= 8 ? 2 : held >= 3 ? 4 : 8;
        // The edit distance's second launch of more than four symbols: the pairs in it have
        // wide scores (unrelated, of 20 letters: 4 096 of 2 000 12.6 ms on four
        // wavefronts, 18.7 on two).  Of four symbols it is as good as always empty, which
        // takes longer with more wavefronts.
        if (x.pass == 1 && x.pen_x == 0 && !x.two_bit) x.waves = std::max(x.waves, 4);
      }
      if (!per_pair) {
        HIP_TRY(ctx, timed_launch(ctx, passes[ip].first, st, [&] { return alnk::launch_search(x, st); }));
      } else {
        for (int32_t k = 0; k < L.count; ++k) {
          x.tasks = dtasks + k;
          x.ntasks = 1;
          HIP_TRY(ctx, alnk::launch_search(x, st));
        }
      }
    }
    return ALN_OK;
  }

  if (sw16) {
    alnk::Sw16Args a16;
    a16.b = bp;
    a16.sc = dsc;
    a16.sc_alphabet = hsc.alphabet;
    a16.ws = ws;
    a16.res = d_res;
    a16.rerun_count = rerun_cnt;
    a16.rerun = rerun_q;
    a16.rerun_threshold = 32767 - std::max(hsc.max_s, 0);
    if (!per_pair) {
      for (const LaunchDesc &L : plan->launches) {
        if (L.kind != K_SW16) continue;
        a16.tasks = reinterpret_cast<const alnk::Sw16Task *>(ws + plan->sw16_off) + L.first;
        a16.ntasks = L.count;
        a16.items = reinterpret_cast<const alnk::Sw16Item *>(ws + plan->sw16_items_off);
        a16.nitems = (int32_t)plan->sw16_items.size();
        a16.wide_both = plan->sw16_both;
        HIP_TRY(ctx, timed_launch(ctx, "sw16", st, [&] {
                  return alnk::launch_sw16(L.rows, a16, st);
                }));
      }
    } else {
      for (size_t k = 0; k < plan->sw16_single.size(); ++k) {
        a16.tasks = reinterpret_cast<const alnk::Sw16Task *>(ws + plan->sw16_single_off) + k;
        a16.ntasks = 1;
        a16.items = nullptr;
        a16.nitems = 0;
        a16.wide_both = 0;
        HIP_TRY(ctx, alnk::launch_sw16(plan->sw16_single_rows[k], a16, st));
      }
    }
    const LaunchDesc &L = plan->rerun;
    alnk::StripArgs sa;
    sa.b = bp;
    sa.tasks = rerun_q;
    sa.ntasks = L.count;
    sa.dyn_ntasks = rerun_cnt;
    sa.mode = L.mode;
    sa.sc = dsc;
    sa.tb = nullptr;
    sa.res = d_res;
    sa.lds_bnd = L.lds_bnd;
    sa.lds_prof = L.lds_prof;
    sa.waves = 1;
    sa.max_n = 0;
    sa.roll_lanes = sa.roll_full = 0;
    HIP_TRY(ctx, timed_launch(ctx, "strip_i32_rerun", st, [&] {
              return alnk::launch_strip(L.rows, L.mode, false, L.small, sa, st);
            }));
    return ALN_OK;
  }

  auto diag_args = [&](const PairTask *tasks, int32_t ntasks, const int32_t *dyn, int widen_rows,
                       int32_t *wcnt, PairTask *wq) {
    alnk::DiagArgs da;
    da.b = bp;
    da.tasks = tasks;
    da.ntasks = ntasks;
    da.dyn_ntasks = dyn;
    da.band_w = plan->p.band_w;
    da.xdrop = plan->p.xdrop;
    da.sc = dsc;
    da.tb = ws + plan->tb_base;
    da.res = d_res;
    da.widen_count = wcnt;
    da.widen = wq;
    da.widen_rows = widen_rows;
    da.match_mismatch = hsc.match_mismatch;
    return da;
  };
  PairTask *wq0 = plan->xdrop ? reinterpret_cast<PairTask *>(ws + plan->widen_off[0]) : nullptr;
  bool zd_lanes = false; // Z-drop on the 64-cell windows of the lanes kernel
  for (const LaunchDesc &L : plan->launches)
    zd_lanes = zd_lanes || (L.kind == K_DIAG && L.sides == 16 && L.window == 64 && plan->p.prune == ALN_ZDROP);
  PairTask *wq1 = plan->xdrop ? reinterpret_cast<PairTask *>(ws + plan->widen_off[1]) : nullptr;
  // diagonals of the longest query and reference: no region is wider
  const int64_t span = (int64_t)plan->max_m + plan->max_n;
  // cells a lane of the first widening pass (see there)
  const int wide_rows = plan->p.prune == ALN_ZDROP && zdrop_within(hsc, plan->p, kZdropReach) ? 8 : 16;
  PairTask *wq2 = plan->xtb_lanes ? reinterpret_cast<PairTask *>(ws + plan->widen_off[2]) : nullptr;
  if (plan->xtb_lanes) {
    // codes from the lanes kernel; pairs whose region outgrows its
    // window are recomputed with codes by the one-side pass (queue 2)
    alnk::XdlArgs xa;
    xa.zdrop = 0;
    xa.lps = plan->xtb_lps;
    xa.window = 64;
    xa.b = bp;
    xa.tasks = dtasks + plan->xtb_first;
    xa.ntasks = plan->xtb_count;
    xa.queue = widen_cnt + 2;
    xa.xdrop = plan->p.xdrop;
    xa.gap_open = hsc.gap_open;
    xa.gap_extend = hsc.gap_extend;
    xa.match = hsc.match;
    xa.mismatch = hsc.mismatch;
    xa.res = d_res;
    xa.widen_count = widen_cnt + 4;
    xa.widen = wq2;
    xa.widen_rows = 4;
    xa.tb = ws + plan->tb_base;
    if (!per_pair) {
      HIP_TRY(ctx, timed_launch(ctx, "xdrop_lanes_tb", st, [&] {
                return alnk::launch_xdrop_lanes(true, xa, plan->xtb_grid, st);
              }));
    } else {
      for (int32_t k = 0; k < plan->xtb_count; ++k) {
        xa.tasks = dtasks + plan->xtb_first + k;
        xa.ntasks = 1;
        HIP_TRY(ctx, alnk::launch_xdrop_lanes(true, xa, 1, st));
      }
    }
    alnk::DiagArgs d = diag_args(wq2, plan->n, widen_cnt + 4, 16, widen_cnt, wq0);
    if (span > 126)
      HIP_TRY(ctx, timed_launch(ctx, "xdrop_tb", st, [&] {
                return alnk::launch_diag(4, ALN_EXTEND, plan->p.prune, true, d, st);
              }));
  } else if (plan->xtb_count > 0) {
    // X-drop / Z-drop with CIGAR: one pass per pair computes the results and
    // writes the traceback codes; regions that outgrow its window go to the
    // widening queue below (score only) and the walk decides their CIGAR
    auto xtb = [&](int32_t first, int32_t count) {
      alnk::DiagArgs d = diag_args(dtasks + first, count, nullptr, wide_rows,
                                   widen_cnt, wq0);
      return alnk::launch_diag(4, ALN_EXTEND, plan->p.prune, true, d, st);
    };
    const char *fam = plan->p.prune == ALN_ZDROP ? "zdrop_tb" : "xdrop_tb";
    if (!per_pair) {
      HIP_TRY(ctx, timed_launch(ctx, fam, st, [&] { return xtb(plan->xtb_first, plan->xtb_count); }));
    } else {
      for (int32_t k = 0; k < plan->xtb_count; ++k) HIP_TRY(ctx, xtb(plan->xtb_first + k, 1));
    }
  }
  for (const LaunchDesc &L : plan->launches) {
    if (L.kind == K_DIAG) {
      if (plan->xtb_count > 0) continue; // the traceback pass above replaces it
      const int widen_rows = plan->xdrop ? (zd_lanes ? 4 : wide_rows) : 0;
      if (L.sides == 16) {
        alnk::XdlArgs xa;
        xa.tb = nullptr;
        xa.zdrop = plan->p.prune == ALN_ZDROP ? 1 : 0;
        xa.lps = L.lps;
        xa.window = L.window;
        xa.b = bp;
        xa.tasks = dtasks + L.first;
        xa.ntasks = L.count;
        xa.queue = widen_cnt + 2;
        xa.xdrop = plan->p.xdrop;
        xa.gap_open = hsc.gap_open;
        xa.gap_extend = hsc.gap_extend;
        xa.match = hsc.match;
        xa.mismatch = hsc.mismatch;
        xa.res = d_res;
        xa.widen_count = widen_cnt;
        xa.widen = wq0;
        xa.widen_rows = widen_rows;
        if (!per_pair) {
          HIP_TRY(ctx, timed_launch(ctx, xa.zdrop ? "zdrop_lanes" : "xdrop_lanes", st, [&] {
                    return alnk::launch_xdrop_lanes(false, xa, L.grid, st);
                  }));
        } else {
          for (int32_t k = 0; k < L.count; ++k) {
            xa.tasks = dtasks + L.first + k;
            xa.ntasks = 1;
            HIP_TRY(ctx, alnk::launch_xdrop_lanes(false, xa, 1, st));
          }
        }
        continue;
      }
      auto go = [&](const alnk::DiagArgs &da) {
        return L.sides == 4 ? alnk::launch_xdrop_group(plan->p.prune, da, st)
                            : alnk::launch_diag(L.rows, L.mode, plan->p.prune, L.tb, da, st);
      };
      if (!per_pair) {
        alnk::DiagArgs da = diag_args(dtasks + L.first, L.count, nullptr, widen_rows, widen_cnt, wq0);
        const char *fam = plan->p.prune == ALN_ZDROP ? "zdrop" : (plan->xdrop ? "xdrop" : "diag_band");
        HIP_TRY(ctx, timed_launch(ctx, fam, st, [&] { return go(da); }));
      } else {
        for (int32_t k = 0; k < L.count; ++k) {
          alnk::DiagArgs da = diag_args(dtasks + L.first + k, 1, nullptr, widen_rows, widen_cnt, wq0);
          HIP_TRY(ctx, go(da));
        }
      }
      continue;
    }
    alnk::StripArgs sa;
    sa.b = bp;
    sa.dyn_ntasks = nullptr;
    sa.mode = L.mode;
    sa.sc = dsc;
    sa.tb = ws + plan->tb_base;
    sa.res = d_res;
    sa.lds_bnd = L.lds_bnd;
    sa.lds_prof = L.lds_prof;
    sa.waves = L.waves;
    sa.max_n = L.max_n;
    sa.band_w = plan->strip_band_w;
    sa.ring_cols = L.lds_bnd / 8;
    sa.roll_lanes = L.kind == K_ROLL ? L.waves : 0;
    sa.roll_full = L.full ? 1 : 0;
    if (L.kind == K_ROLL) sa.band_w = L.full ? 1 << 28 : plan->p.band_w;
    const char *const bfam = L.kind == K_ROLL ? (L.full ? "roll_i32" : "band_roll") : "band_strip";
    if (L.kind == K_BAND || L.kind == K_ROLL) {
      if (!per_pair) {
        sa.tasks = dtasks + L.first;
        sa.ntasks = L.count;
        HIP_TRY(ctx, timed_launch(ctx, bfam, st, [&] {
                  return alnk::launch_band_strip(L.rows, L.mode, L.tb, L.small, sa, st);
                }));
      } else {
        for (int32_t k = 0; k < L.count; ++k) {
          sa.tasks = dtasks + L.first + k;
          sa.ntasks = 1;
          HIP_TRY(ctx, alnk::launch_band_strip(L.rows, L.mode, L.tb, L.small, sa, st));
        }
      }
      continue;
    }
    if (!per_pair) {
      sa.tasks = dtasks + L.first;
      sa.ntasks = L.count;
      HIP_TRY(ctx, timed_launch(ctx, "strip_i32", st, [&] {
                return alnk::launch_strip(L.rows, L.mode, L.tb, L.small, sa, st);
              }));
    } else {
      for (int32_t k = 0; k < L.count; ++k) {
        sa.tasks = dtasks + L.first + k;
        sa.ntasks = 1;
        HIP_TRY(ctx, alnk::launch_strip(L.rows, L.mode, L.tb, L.small, sa, st));
      }
    }
  }
  if (plan->xdrop) {
    // Pairs whose surviving region outgrew their window, in wider ones.  A
    // handful of long sides sets each pass's time, one wavefront each: Z-drop
    // regions that Z keeps within 180 diagonals of the best cell's seldom pass 512, where an
    // antidiagonal takes two thirds of the 1024-diagonal kernel's (25 000 sides at Z = 100:
    // 6.4 against 9.5 ms), so that comes first; from the 64-cell lanes form even
    // 256 diagonals hold most.  Past that line both passes would be run for many: 3 000 sides of
    // 2 500 bp, e = -2, ms without / with 512, Z = 180 8.2 / 5.3, Z = 240 5.5 / 8.1; 2 000 at Z =
    // 300 6.5 / 12.1; 20 000 at e = -1, Z = 100 50.3 / 66.5.
    const int pr = plan->p.prune;
    const char *fam = pr == ALN_ZDROP ? "zdrop_wide" : "xdrop_wide";
    int rows[4] = {16, 32, 0, 0};
    if (wide_rows == 8) {
      rows[0] = zd_lanes ? 4 : 8;
      rows[1] = zd_lanes ? 8 : 16;
      rows[2] = 32;
    }
    // Only the passes that some region of these lengths could need (the windows hold
    // 126 diagonals in 64 cells, else 64 rows - 6; an empty pass takes 2 us).
    int64_t held = plan->xtb_count > 0 ? 250 : INT64_MAX;
    for (const LaunchDesc &L : plan->launches)
      if (L.kind == K_DIAG && plan->xtb_count == 0)
        held = std::min<int64_t>(held, L.sides == 16 ? (L.window == 64 ? 126 : 250)
                                                     : (L.sides == 4 ? 100 : 64 * L.rows - 6));
    for (int k = 0; k < 4 && rows[k]; ++k) {
      if (span <= held) {
        rows[k] = 0;
        break;
      }
      held = 64 * rows[k] - 6;
    }
    int32_t *const cnt[3] = {widen_cnt, widen_cnt + 1, widen_cnt + 4};
    PairTask *const wq[3] = {wq0, wq1, wq0}; // the first queue is read out before it is filled again
    for (int k = 0; rows[k]; ++k) {
      const bool last = rows[k + 1] == 0;
      alnk::DiagArgs d = diag_args(wq[k], plan->n, cnt[k], rows[k + 1], last ? nullptr : cnt[k + 1],
                                   last ? nullptr : wq[k + 1]);
      HIP_TRY(ctx, timed_launch(ctx, fam, st, [&] {
                return alnk::launch_diag(rows[k], ALN_EXTEND, pr, false, d, st);
              }));
    }
  }
  if (plan->p.want_cigar) {
    alnk::WalkArgs wa;
    wa.b = bp;
    wa.mode = plan->p.mode;
    wa.layout = 0;
    wa.shares = 1;
    wa.diag_stride = plan->xtb_lanes ? 1 : (plan->xtb_count > 0 ? 2 : 8);
    wa.dyn_ntasks = nullptr;
    wa.band_w = plan->p.band_w;
    wa.sc = dsc;
    wa.tb = ws + plan->tb_base;
    wa.res = d_res;
    wa.cigar = d_cigar;
    auto walk = [&](int layout, const PairTask *tasks, int32_t nt) -> hipError_t {
      wa.tasks = tasks;
      wa.ntasks = nt;
      wa.layout = layout;
      wa.band_w = layout >= 2 ? plan->strip_band_w : plan->p.band_w;
      // (LOCAL paths start at no row known; full-matrix rolling blocks are short)
      const bool one = layout < 2 || plan->p.mode == ALN_LOCAL || (layout == 3 && plan->roll_full_tb);
      wa.shares = one ? 1 : walk_shares(ctx, nt, plan->max_m);
      return layout == 1 ? alnk::launch_walk_diag(wa, st) : alnk::launch_walk(layout, wa, st);
    };
    if (!per_pair) {
      HIP_TRY(ctx, timed_launch(ctx, "walk", st, [&] { return walk(0, dtasks, plan->n_strip_tb); }));
      HIP_TRY(ctx, timed_launch(ctx, "walk", st, [&] {
                return walk(1, dtasks + plan->first_diag_tb, plan->n_diag_tb);
              }));
      HIP_TRY(ctx, timed_launch(ctx, "walk", st, [&] {
                return walk(2, dtasks + plan->first_band_tb, plan->n_band_tb);
              }));
      HIP_TRY(ctx, timed_launch(ctx, "walk", st, [&] {
                return walk(3, dtasks + plan->first_roll_tb, plan->n_roll_tb);
              }));
    } else {
      for (int32_t k = 0; k < plan->n_strip_tb; ++k) HIP_TRY(ctx, walk(0, dtasks + k, 1));
      for (int32_t k = 0; k < plan->n_diag_tb; ++k)
        HIP_TRY(ctx, walk(1, dtasks + plan->first_diag_tb + k, 1));
      for (int32_t k = 0; k < plan->n_band_tb; ++k)
        HIP_TRY(ctx, walk(2, dtasks + plan->first_band_tb + k, 1));
      for (int32_t k = 0; k < plan->n_roll_tb; ++k)
        HIP_TRY(ctx, walk(3, dtasks + plan->first_roll_tb + k, 1));
    }
    if (plan->xtb_lanes) { // the pairs the one-side pass recomputed, in its layout
      wa.diag_stride = 2;
      wa.dyn_ntasks = widen_cnt + 4;
      HIP_TRY(ctx, timed_launch(ctx, "walk", st, [&] { return walk(1, wq2, plan->n); }));
    }
  }
  return ALN_OK;
}

aln_status aln_execute(aln_ctx *ctx, aln_plan *plan, const aln_batch *batch, void *d_ws,
                       uint64_t ws_bytes, aln_result *d_res, uint32_t *d_cigar,
                       uint64_t cigar_words, void *stream) {
  aln_status st = exec_check(ctx, plan, batch, d_ws, ws_bytes, d_res, d_cigar, cigar_words);
  if (st != ALN_OK) return st;
  return run_plan(ctx, plan, batch, d_ws, d_res, d_cigar, (hipStream_t)stream, false);
}

aln_status aln_execute_per_pair(aln_ctx *ctx, aln_plan *plan, const aln_batch *batch, void *d_ws,
                                uint64_t ws_bytes, aln_result *d_res, uint32_t *d_cigar,
                                uint64_t cigar_words, void *stream) {
  aln_status st = exec_check(ctx, plan, batch, d_ws, ws_bytes, d_res, d_cigar, cigar_words);
  if (st != ALN_OK) return st;
  return run_plan(ctx, plan, batch, d_ws, d_res, d_cigar, (hipStream_t)stream, true);
}

aln_status aln_graph_capture(aln_ctx *ctx, aln_plan *plan, const aln_batch *batch, void *d_ws,
                             uint64_t ws_bytes, aln_result *d_res, uint32_t *d_cigar,
                             uint64_t cigar_words, void *stream) {
  aln_status st = exec_check(ctx, plan, batch, d_ws, ws_bytes, d_res, d_cigar, cigar_words);
  if (st != ALN_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  if (s == nullptr) return fail(ctx, ALN_E_INVAL, "graph capture needs a non-default stream");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  if (plan->gexec) {
    (void)hipGraphExecDestroy(plan->gexec);
    plan->gexec = nullptr;
  }
  if (plan->graph) {
    (void)hipGraphDestroy(plan->graph);
    plan->graph = nullptr;
  }
  HIP_TRY(ctx, hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
  st = run_plan(ctx, plan, batch, d_ws, d_res, d_cigar, s, false);
  hipGraph_t g = nullptr;
  hipError_t e = hipStreamEndCapture(s, &g);
  if (st != ALN_OK) {
    if (g) (void)hipGraphDestroy(g);
    return st;
  }
  if (e != hipSuccess) return fail(ctx, ALN_E_DEVICE, "end capture: %s", hipGetErrorString(e));
  plan->graph = g;
  HIP_TRY(ctx, hipGraphInstantiate(&plan->gexec, g, nullptr, nullptr, 0));
  HIP_TRY(ctx, hipGraphLaunch(plan->gexec, s));
  return ALN_OK;
}

int64_t aln_plan_describe(const aln_plan *plan, aln_launch_info *launches, int32_t max_launches,
                          int32_t *n_launches, aln_task_info *tasks, int64_t max_tasks) {
  if (!plan || max_launches < 0 || max_tasks < 0) return ALN_E_INVAL;
  int32_t nl = 0;
  int64_t nt = 0;
  auto add_launch = [&](const char *fam, int tile, int sides, int64_t first, int64_t count) {
    if (launches && nl < max_launches) {
      aln_launch_info &L = launches[nl];
      memset(&L, 0, sizeof L);
      std::snprintf(L.family, sizeof L.family, "%s", fam);
      L.tile = tile;
      L.sides = sides;
      L.first = (int32_t)first;
      L.count = (int32_t)count;
    }
    ++nl;
  };
  auto add_task = [&](int32_t launch, int32_t pair, int64_t tb_off, int64_t tb_bytes,
                      int64_t cigar_off, int32_t cigar_cap, int32_t tile) {
    if (tasks && nt < max_tasks) {
      aln_task_info &T = tasks[nt];
      T.launch = launch;
      T.pair = pair;
      T.tb_off = tb_off;
      T.tb_bytes = tb_bytes;
      T.cigar_off = cigar_off;
      T.cigar_cap = cigar_cap;
      T.tile = tile;
    }
    ++nt;
  };
  // traceback bytes of a task: up to the next reservation (offsets grow in
  // task order), the last up to the end of the traceback area
  std::vector<int64_t> tb_end(plan->tasks.size(), (int64_t)plan->tb_bytes);
  {
    int64_t next = (int64_t)plan->tb_bytes;
    for (size_t k = plan->tasks.size(); k-- > 0;) {
      if (plan->tasks[k].tb_off >= 0) {
        tb_end[k] = next;
        next = plan->tasks[k].tb_off;
      }
    }
  }
  auto pair_tasks = [&](int32_t launch, int64_t first, int64_t count) {
    for (int64_t k = first; k < first + count; ++k) {
      const alnk::PairTask &t = plan->tasks[(size_t)k];
      const bool tb = t.tb_off >= 0 && plan->p.want_cigar;
      add_task(launch, t.pair, tb ? t.tb_off : -1, tb ? tb_end[(size_t)k] - t.tb_off : 0,
               plan->p.want_cigar ? t.cigar_off : -1, plan->p.want_cigar ? t.cigar_cap : 0, t.rows);
    }
  };
  if (plan->fold) {
    for (const auto &F : plan->fold_launches) {
      const int32_t id = nl;
      add_launch("fold", F.stride, F.elt, F.first, F.count);
      for (int32_t k = F.first; k < F.first + F.count; ++k)
        add_task(id, plan->fold_tasks[(size_t)k].seq, -1, 0, -1, 0, F.stride);
    }
  } else if (plan->xtb_count > 0) {
    const int32_t id = nl;
    const char *fam = plan->xtb_lanes ? "xdrop_lanes_tb"
                                      : (plan->p.prune == ALN_ZDROP ? "zdrop_tb" : "xdrop_tb");
    add_launch(fam, 4, plan->xtb_lanes ? 64 / plan->xtb_lps : 1, plan->xtb_first, plan->xtb_count);
    pair_tasks(id, plan->xtb_first, plan->xtb_count);
  } else {
    for (const LaunchDesc &L : plan->launches) {
      const int32_t id = nl;
      if (L.kind == K_SW16) {
        add_launch("sw16", L.rows, 2, L.first, L.count);
        for (int32_t k = L.first; k < L.first + L.count; ++k) {
          const alnk::Sw16Task &t = plan->sw16_tasks[(size_t)k];
          add_task(id, t.pa, -1, 0, -1, 0, L.rows);
          if (t.pb >= 0) add_task(id, t.pb, -1, 0, -1, 0, L.rows);
        }
        continue;
      }
      const char *fam = "strip_i32";
      if (L.kind == K_SEARCH) fam = L.pen_x > 0 ? "search_affine" : "search";
      if (L.kind == K_BAND) fam = "band_strip";
      if (L.kind == K_ROLL) fam = L.full ? "roll_i32" : "band_roll";
      if (L.kind == K_DIAG) {
        if (plan->p.prune == ALN_BAND) fam = "diag_band";
        else if (plan->p.prune == ALN_ZDROP)
          fam = L.sides == 16 ? "zdrop_lanes" : (L.sides == 4 ? "zdrop_group" : "zdrop");
        else fam = L.sides == 16 ? "xdrop_lanes" : (L.sides == 4 ? "xdrop_group" : "xdrop");
      }
      add_launch(fam, L.rows,
                 (L.kind == K_STRIP || L.kind == K_BAND) ? L.waves
                 : L.kind == K_ROLL ? 64 / L.waves : (L.sides == 16 ? 64 / L.lps : L.sides), L.first,
                 L.count);
      pair_tasks(id, L.first, L.count);
    }
  }
  if (n_launches) *n_launches = nl;
  return nt;
}

aln_status aln_graph_launch(aln_ctx *ctx, aln_plan *plan, void *stream) {
  if (!ctx || !plan || !plan->gexec) return fail(ctx, ALN_E_INVAL, "no captured graph");
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  HIP_TRY(ctx, hipGraphLaunch(plan->gexec, (hipStream_t)stream));
  return ALN_OK;
}

} // extern "C"

aln_status alnrt::plan_run(aln_ctx *ctx, aln_plan *plan, const aln_batch *b, void *d_ws,
                           aln_result *d_res, uint32_t *d_cigar, hipStream_t st, bool per_pair) {
  return run_plan(ctx, plan, b, d_ws, d_res, d_cigar, st, per_pair);
}

// ------------------------------------------------------------------ folding

extern "C" {

aln_status aln_fold_plan_create(aln_ctx *ctx, const aln_fold_params *params, int32_t n,
                                const int32_t *len_host, aln_plan **plan, aln_footprint *fp) {
  if (!ctx || !params || !plan || n < 0 || (n > 0 && !len_host))
    return fail(ctx, ALN_E_INVAL, "null argument or negative n");
  *plan = nullptr;
  const aln_fold_params &p = *params;
  int maxpair = 0;
  for (int k = 0; k < 16; ++k) {
    if (p.pair[k] < 0 || p.pair[k] > 127) return fail(ctx, ALN_E_INVAL, "pair scores must be 0..127");
    maxpair = std::max(maxpair, p.pair[k]);
  }
  if (p.min_loop < 0 || p.warmup < 0) return fail(ctx, ALN_E_INVAL, "min_loop and warmup >= 0");
  if (p.block != 0 && p.block != 256 && p.block != 512 && p.block != 1024)
    return fail(ctx, ALN_E_INVAL, "block must be 0, 256, 512 or 1024");
  // LDS of one CU, less the kernel's few static words
  const int64_t lds_max = std::min<int64_t>(ctx->lds_per_cu, 160 * 1024) - 256;
  // Per sequence: the row stride of its folded triangle (the smallest of
  // kFoldStrides above its length) and the element width (one byte when
  // every score fits 0..253 -- 255 marks minus infinity -- else two).
  struct Cls {
    int elt, stride;
  };
  std::vector<Cls> cls(n);
  for (int32_t s = 0; s < n; ++s) {
    const int32_t L = len_host[s];
    if (L < 0) return fail(ctx, ALN_E_INVAL, "negative length");
    int stride = 0;
    for (int sc : alnk::kFoldStrides)
      if (L + 1 <= sc) {
        stride = sc;
        break;
      }
    const int64_t maxF = (int64_t)maxpair * (L / 2);
    const bool u8 = stride && maxF <= 253 && (int64_t)alnk::fold_lds_bytes(1, stride, L) <= lds_max;
    const bool i16 =
        stride && maxF <= 32767 && (int64_t)alnk::fold_lds_bytes(2, stride, L) <= lds_max;
    if (!u8 && !i16)
      return fail(ctx, ALN_E_UNSUPPORTED,
                  "sequence %d (%d nt): longer than 511, or its triangle does not fit LDS, or "
                  "its scores could exceed 32767", s, L);
    cls[s] = Cls{u8 ? 1 : 2, stride};
  }
  aln_plan *pl = new (std::nothrow) aln_plan;
  if (!pl) return fail(ctx, ALN_E_NOMEM, "plan allocation");
  pl->ctx = ctx;
  pl->n = n;
  pl->fold = true;
  pl->fold_p = p;
  pl->qlen.assign(len_host, len_host + n);
  int64_t cells = 0;
  auto add_launch = [&](const std::vector<int32_t> &idx, int elt, int stride, int block) {
    aln_plan::FoldLaunch L;
    L.elt = elt;
    L.stride = stride;
    L.block = p.block ? p.block : block;
    L.first = (int32_t)pl->fold_tasks.size();
    L.count = (int32_t)idx.size();
    L.max_n = 0;
    for (int32_t s : idx) {
      L.max_n = std::max(L.max_n, len_host[s]);
      pl->fold_tasks.push_back(alnk::FoldTask{s, len_host[s]});
      cells += (int64_t)len_host[s] * (len_host[s] - 1) / 2;
    }
    pl->fold_launches.push_back(L);
  };
  auto longer = [&](int32_t x, int32_t y) { return len_host[x] > len_host[y]; };
  // Unpruned with byte scores (tiles), the longest sequence first (LPT): one launch of
  // those too long for two workgroups a CU (368 nt and more), whose last round
  // leaves CUs idle, so shorter ones follow in it as long as it does not end later
  // (its course is followed here with the time of a workgroup alone on its CU, us);
  // and one launch of the rest, two or more workgroups a CU.  2 048 sequences of
  // 76..500 nt, before the products of 0 / 1 scores went to the matrix cores: four
  // launches by length (LDS of 128, 256, 384, 512 nt) 1 493 us, these two 1 246, with the
  // gaps filled 1 143; a third launch for those of which eight share a CU 1 170.
  // Wavefronts a workgroup, by how many share a CU, 4 / 8 / 16, 2 048 of 500 nt: 3.10 /
  // 2.38 / 2.29 ms, of 300 nt 0.71 / 0.66 / 1.01, of 180 nt 0.21 / 0.32 / 0.56.
  const bool tiles = p.xdrop < 0;
  if (tiles) {
    auto per_cu = [&](int32_t s) {
      return lds_max / (int64_t)alnk::fold_tile_lds_bytes(len_host[s], 4);
    };
    auto us = [&](int32_t s) {
      const double L = len_host[s];
      return 0.36 * L + (maxpair <= 1 ? 0.9e-6 : 1.8e-6) * L * L * L;
    };
    std::vector<int32_t> idx, alone, shared;
    for (int32_t s = 0; s < n; ++s)
      if (cls[s].elt == 1) idx.push_back(s);
    std::stable_sort(idx.begin(), idx.end(), longer);
    const size_t cus = (size_t)ctx->cus;
    std::vector<double> busy; // until when each CU is, a min heap
    auto give = [&](int32_t s) {
      if (busy.size() < cus) {
        busy.push_back(us(s));
      } else {
        std::pop_heap(busy.begin(), busy.end(), std::greater<double>());
        busy.back() += us(s);
      }
      std::push_heap(busy.begin(), busy.end(), std::greater<double>());
      alone.push_back(s);
    };
    size_t k = 0;
    for (; k < idx.size() && per_cu(idx[k]) < 2; ++k) give(idx[k]);
    const double end = busy.empty() ? 0 : *std::max_element(busy.begin(), busy.end());
    for (; k < idx.size(); ++k) {
      const double from = busy.size() < cus ? 0 : busy.front();
      if (from + us(idx[k]) <= end) give(idx[k]);
      else shared.push_back(idx[k]);
    }
    for (const auto *g : {&alone, &shared}) {
      if (g->empty()) continue;
      const int64_t share = per_cu((*g)[0]);
      add_launch(*g, 1, 16 * alnk::fold_tile_rows(len_host[(*g)[0]]),
                 share >= 3 ? 256 : (share == 2 ? 512 : 1024));
    }
  }
  // The other forms: one launch per (stride, width), the widest rows first;
  // within a launch the longest sequence first.  Threads per workgroup so that the
  // workgroups LDS lets share a CU hold about 16 wavefronts.
  for (int si = 3; si >= 0; --si) {
    for (int elt = 2; elt >= (tiles ? 2 : 1); --elt) {
      const int stride = alnk::kFoldStrides[si];
      std::vector<int32_t> idx;
      for (int32_t s = 0; s < n; ++s)
        if (cls[s].stride == stride && cls[s].elt == elt) idx.push_back(s);
      if (idx.empty()) continue;
      std::stable_sort(idx.begin(), idx.end(), longer);
      const int64_t lds = (int64_t)alnk::fold_lds_bytes(elt, stride, len_host[idx[0]]);
      const int64_t per_cu = std::max<int64_t>(1, lds_max / std::max<int64_t>(lds, 1));
      add_launch(idx, elt, stride, per_cu >= 4 ? 256 : (per_cu >= 2 ? 512 : 1024));
    }
  }
  pl->upload_bytes = sizeof(alnk::FoldTask) * pl->fold_tasks.size();
  pl->tasks_bytes = align_up(std::max<uint64_t>(pl->upload_bytes, 1));
  pl->ws_bytes = pl->tasks_bytes;
  pl->cells = cells;
  if (alnrt::plan_alloc_staging(pl) != ALN_OK) {
    delete pl;
    return fail(ctx, ALN_E_NOMEM, "staging");
  }
  plan_stage(pl, pl->pinned);
  if (fp) {
    fp->workspace_bytes = pl->ws_bytes;
    fp->traceback_bytes = 0;
    fp->cigar_words = 0;
    fp->cells = cells;
  }
  *plan = pl;
  return ALN_OK;
}

aln_status aln_fold_execute(aln_ctx *ctx, aln_plan *plan, const aln_fold_batch *b, void *d_ws,
                            uint64_t ws_bytes, aln_fold_result *d_res, void *stream) {
  if (!ctx || !plan || !b || plan->ctx != ctx || !plan->fold)
    return fail(ctx, ALN_E_INVAL, "bad context or folding plan");
  if (b->n != plan->n) return fail(ctx, ALN_E_INVAL, "batch has %d sequences, plan %d", b->n, plan->n);
  if (plan->n == 0) return ALN_OK;
  if (!d_res || !b->x || !b->off || !b->len) return fail(ctx, ALN_E_INVAL, "null device pointer");
  if (!d_ws || ws_bytes < plan->ws_bytes)
    return fail(ctx, ALN_E_CAPACITY, "workspace %llu < %llu bytes", (unsigned long long)ws_bytes,
                (unsigned long long)plan->ws_bytes);
  if (ctx->device < 0) return fail(ctx, ALN_E_DEVICE, "the context has no device");
  hipStream_t st = (hipStream_t)stream;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  HIP_TRY(ctx, hipMemcpyAsync(d_ws, plan->pinned, plan->upload_bytes, hipMemcpyHostToDevice, st));
  alnk::FoldArgs a;
  a.x = b->x;
  a.off = b->off;
  a.len = b->len;
  for (int k = 0; k < 16; ++k) a.pair[k] = plan->fold_p.pair[k];
  a.min_loop = plan->fold_p.min_loop;
  a.xdrop = plan->fold_p.xdrop;
  a.warmup = plan->fold_p.warmup;
  a.res = d_res;
  const alnk::FoldTask *tasks = static_cast<const alnk::FoldTask *>(d_ws);
  for (const aln_plan::FoldLaunch &L : plan->fold_launches) {
    a.tasks = tasks + L.first;
    a.ntasks = L.count;
    a.max_n = L.max_n;
    HIP_TRY(ctx, timed_launch(ctx, "fold", st, [&] {
              return alnk::launch_fold(L.elt, L.block, L.stride, a, st);
            }));
  }
  return ALN_OK;
}

} // extern "C"
