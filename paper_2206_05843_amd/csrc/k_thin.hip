// Thin-run solve kernels: level-by-level forward substitution (Sec. II.A,
// Algorithm 1) over the level-ordered copy of L, or of the rewritten L'
// (Sec. II.B) after the b-transform b' = T b (applied before the level chain
// starts, since it does not depend on x). Wide levels are in k_wide.hip.
//
// Work vectors are permuted to level order and RHS-interleaved: entry (pos, c)
// of bp/xp is at pos*nrhs + c, so the rows of one level are contiguous and one
// row's right-hand sides share cache lines.
//
// Two schedules per level:
//  * thin runs: consecutive narrow levels in LDS windows, each solved by one
//    workgroup, whose levels are separated by workgroup barriers or by nothing
//    (no device-wide synchronisation). Values a window produces are kept in LDS,
//    where its later levels read them, and go to global memory for the windows
//    after it, which one workgroup solves in turn or, spread over workgroups, as
//    the values they read become final.
//  * wide levels: one launch over the device per level (kernel boundaries order
//    the levels).
#include <algorithm>

#include "common.h"
#include "sync.h"
#include "wait.h"

namespace {

constexpr int kWinBytes = 159 * 1024;  // dynamic LDS of a thin-run workgroup (of the CU's 160 KB)
// Its first 16 bytes hold control words (no static LDS in these kernels: it
// would offset the dynamic region and misalign its 16-byte records); the
// window layout starts after them.
constexpr int kCtlBytes = 16;
struct Ctl {
  int32_t next;  // batched launch: the workgroup's next queue ticket
  int32_t pad[3];
};


// A thin run is cut into LDS windows (consecutive levels, chosen on the host so
// that the window's rows and dependency records fit in LDS). Per window:
//  phase 1 (all rows in parallel): the window's static image, built once per
//    schedule, is streamed into LDS: per row its first K in-window
//    dependencies (weights and slots; absent ones point to a zero entry with
//    weight 0, so phase 2 needs no predication), its diagonal with the
//    reciprocal, and a list of {weight, slot} records for the dependencies
//    beyond K. Meanwhile each thread loads, for several rows at once, b' and
//    the row's range of dependencies on earlier windows, then forms
//    v = b' - sum of L(pos,k) x(k) over those (final values, read from global
//    memory, in the row's order);
//  phase 2 (level by level): x = (v - sum over in-window dependencies) / d, in
//    LDS only;
//  then the window's x goes to global memory in one coalesced pass (where the
//    finiteness check happens too), before the next window reads it.
// Rows are in ascending position, so the earlier windows' dependencies come
// first whatever the cut, and the sums and quotients are those of the other
// one-lane executors bit for bit (rows kept in column order excepted).
// A level of phase 2 waits for the x of the level before, and a single wave
// issues an instruction every four or five cycles, so what a level costs is one
// LDS round trip and its instructions. All of a row's x (K inline dependencies)
// are requested at once and the next level's records behind them; a record has
// one address; lanes past the level's end repeat its last row instead of being
// masked (with one column: its owner is then in the same wave and writes the same
// value; with several columns a row's items may lie in two waves, one of which
// could read the partial sum after the other wrote x over it, so there such
// lanes write nothing); waves without a row of the level go straight to the barrier. K is the
// window's width class: 2, 6 or 10 (cut_windows has the rule).
// Levels' records are requested one level ahead and the level bounds read from
// registers when every level of the window has at most one item per thread.
// Windows whose levels have at most 64 items run phase 2 on one wave without
// workgroup barriers.
// Measured (one right-hand side): a 2,000-row window matrix, 277 levels of five
// dependencies a row, 49 us a solve against 95 with two inline dependencies,
// the others in records read two dependent round trips per four, and sections
// with addresses of their own (about 110 and 280 ns a level); the 2D stencil's
// 4,602 levels 888 us against 1,130, its rewritten form 2.69 ms against 2.95.
// win[i] = {first level, flags}; the run's last entry holds the end level.
// kTime (used only to label levels for the learned policy): kDurations: thread 0
// stamps the device wall clock around every level and writes per-level times
// (ns); kFinish: it records the clock at the end of every level, the latest over
// the columns.
enum TimeKind { kNoTimes, kDurations, kFinish };
struct Times {
  float *ns;                   // kDurations, per level
  float ns_per_tick;
  unsigned long long *finish;  // kFinish, per level, then the earliest of level 0
  int32_t nlev;
};
constexpr int kBatch = 4;

// x of a row not yet solved, where other workgroups wait for it: a signalling
// NaN that arithmetic never produces.
__device__ __forceinline__ bool is_pending(double x) {
  return (unsigned long long)__double_as_longlong(x) == kPendingX;
}

// LDS by byte address: these kernels have no static LDS, so their dynamic LDS
// starts at address 0 and an item's address needs no base added to it.
typedef __attribute__((address_space(3))) double lds_f64;
typedef __attribute__((address_space(3))) const uint32_t lds_u32;
__device__ __forceinline__ lds_f64 *lds_d(uint32_t byte) { return (lds_f64 *)(uintptr_t)byte; }
__device__ __forceinline__ uint32_t lds_u(uint32_t byte) { return *(lds_u32 *)(uintptr_t)byte; }

// A window in LDS (byte addresses). v, the partial sums and then x, comes
// first, at kCtlBytes: [(R + 1) * gw] doubles, row R zero; then the row
// records, the overflow records and the level bounds.
struct Win {
  uint32_t rec, ovf;
  const int32_t *lv;   // [NL + 2] level bounds from the window's first position (the last one twice)
  int32_t NL, gw;
};

// acc - sum_j w_j x over n overflow records from record ob on, in order, in
// batches of 4 (tail clamped to a valid record); c8: the column's byte offset.
__device__ __forceinline__ double ovf_sum(const Win &W, double acc, int32_t ob, int32_t n, uint32_t c8) {
  const uint32_t d = W.ovf + 16u * (uint32_t)ob;
  for (int32_t i0 = 0; i0 < n; i0 += kBatch) {
    const int32_t cnt = n - i0;
    double w[kBatch], xv[kBatch];
    uint32_t e[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const uint32_t at = d + 16u * (uint32_t)(i0 + (j < cnt ? j : 0));
      w[j] = *lds_d(at);
      e[j] = lds_u(at + 8);
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) xv[j] = *lds_d(8u * e[j] + c8 + kCtlBytes);
#pragma unroll
    for (int j = 0; j < kBatch; ++j) acc = j < cnt ? fma(-w[j], xv[j], acc) : acc;
  }
  return acc;
}

// The static inputs of one (row, rhs) item in phase 2: its record, its partial
// sum and where its x goes (the packed fields are unpacked where they are used).
template <int K>
struct Item {
  double acc, d, r;
  double w[K > 0 ? K : 1];
  uint32_t ix[K > 0 ? K / 2 + 1 : 1];
  uint32_t at;
  bool own;  // several columns: not a repeat of another lane's item
};

template <int K, int kGw>
__device__ __forceinline__ void load_item(const Win &W, int32_t row, uint32_t c8, Item<K> &it) {
  const uint32_t gw = kGw > 0 ? kGw : W.gw;
  constexpr int kBytes = row_record_bytes(K == 2 ? 0 : K == 6 ? 1 : K == 10 ? 2 : 3);
  const uint32_t rec = __umul24((uint32_t)row, kBytes) + W.rec;
  if constexpr (K > 0) {
#pragma unroll
    for (int j = 0; j < K / 2 + 1; ++j) it.ix[j] = lds_u(rec + 8 * (K + 2) + 4 * j);
#pragma unroll
    for (int j = 0; j < K; ++j) it.w[j] = *lds_d(rec + 8 * j);
  }
  it.d = *lds_d(rec + 8 * K);
  it.r = *lds_d(rec + 8 * (K + 1));
  it.at = kGw == 1 ? 8u * (uint32_t)row : __umul24((uint32_t)row, 8u * gw) + c8;
  it.acc = *lds_d(it.at + kCtlBytes);
}

// The x an item reads, all requested at once. Slots hold byte offsets of one
// column's x, or (several columns) counts of doubles.
template <int K, int kGw>
__device__ __forceinline__ void load_x(const Item<K> &it, uint32_t c8, double (&xv)[K > 0 ? K : 1]) {
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const uint32_t s = j & 1 ? it.ix[j >> 1] >> 16 : it.ix[j >> 1] & 0xffffu;
    xv[j] = *lds_d((kGw == 1 ? s : 8u * s + c8) + kCtlBytes);
  }
}

template <int K, int kGw, bool kOvf>
__device__ __forceinline__ double solve_item(const Win &W, const Item<K> &it, uint32_t c8,
                                             const double (&xv)[K > 0 ? K : 1]) {
  double acc = it.acc;
  if constexpr (K > 0) {
#pragma unroll
    for (int j = 0; j < K; ++j) acc = fma(-it.w[j], xv[j], acc);
    if constexpr (kOvf) {
      const int32_t cnt = (int32_t)(it.ix[K / 2] & 0xffffu), ob = (int32_t)(it.ix[K / 2] >> 16);
      if (cnt > K) acc = ovf_sum(W, acc, ob, cnt - K, kGw == 1 ? 0u : c8);
    }
  }
  return div_by(acc, it.d, it.r);
}

// An x that other workgroups of the launch read: device-coherent.
__device__ __forceinline__ void put_x(double *p, double x) {
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), (unsigned long long)__double_as_longlong(x),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Phase 2 of a window of width K (flags as in the window table). kOvf: the
// window has overflow records. kOneWave: every level has at most 64 items and
// the calling wave solves them all. kNow: an x also goes to global memory as it
// is solved, to byte gmul times its place in the window behind gx, for the
// workgroups that wait for it. tid: the thread's number, counted from the first
// wave to work.
template <int WG, int kGw, int K, bool kOvf, bool kOneWave, int kTime, bool kNow>
__device__ __forceinline__ void solve_levels(const Win &W, int32_t flags, int32_t lA, const Times &T,
                                             unsigned long long t_prev, float p1_per_row, double *gx, uint32_t gmul,
                                             int tid) {
  constexpr bool kOne = kGw == 1;
  const int32_t gw = kGw > 0 ? kGw : W.gw;
  const int32_t *lv = W.lv;
  auto put = [&](uint32_t at, double x) {
    *lds_d(at + kCtlBytes) = x;
    if constexpr (kNow) put_x(reinterpret_cast<double *>(reinterpret_cast<char *>(gx) + (uint64_t)at * gmul), x);
  };
  auto stamp = [&](int32_t lg) {
    if (kTime != kNoTimes && tid == 0) {
      const unsigned long long now = wall_clock64();
      if (kTime == kDurations) {
        T.ns[lA + lg] = (float)(now - t_prev) * T.ns_per_tick + p1_per_row * (float)(lv[lg + 1] - lv[lg]);
        t_prev = now;
      } else {
        atomicMax(T.finish + lA + lg, now);
        if (lA + lg == 0) atomicMin(T.finish + T.nlev, now);
      }
    }
  };
  if (kOneWave || (flags & 2)) {
    // one item per thread: row s0 of the level, column c8 / 8
    const int32_t s0 = kOne ? tid : tid / gw;
    const uint32_t c8 = kOne ? 0u : 8u * (uint32_t)(tid - s0 * gw);
    const int32_t wave0 = kOneWave ? 0 : __builtin_amdgcn_readfirstlane((kOne ? (tid & ~63) : (tid & ~63) / gw));
    const int lane = tid & 63;
    // levels in chunks of 62: lane i holds the bound of level l0 + i, read
    // once per chunk, so a level's bounds come from registers; the level past
    // a chunk's (or the window's) end is loaded and dropped
    constexpr int kChunk = 62;
    for (int32_t l0 = 0; l0 < W.NL; l0 += kChunk) {
      const int32_t nlc = W.NL - l0 < kChunk ? W.NL - l0 : kChunk;
      const int32_t lvreg = lv[l0 + lane <= W.NL ? l0 + lane : W.NL];
      int32_t pb = __builtin_amdgcn_readlane(lvreg, 0), pe = __builtin_amdgcn_readlane(lvreg, 1);
      bool on = kOneWave || wave0 < pe - pb;
      bool wide = !kOneWave && (pe - pb) * gw > 64;
      Item<K> a, b;
      auto load = [&](Item<K> &it) {
        load_item<K, kGw>(W, min(pb + s0, pe - 1), c8, it);
        if constexpr (!kOne) it.own = pb + s0 < pe;
      };
      if (on) load(a);
      auto step = [&](int32_t l, Item<K> &cur, Item<K> &nxt) {
        // the level's x first, then the next level's records, which do not
        // depend on it (LDS returns in order)
        double xv[K > 0 ? K : 1];
        if (on) load_x<K, kGw>(cur, c8, xv);
        pb = pe;
        pe = __builtin_amdgcn_readlane(lvreg, l + 2);
        const bool on_next = kOneWave || wave0 < pe - pb;
        if (on_next) load(nxt);
        __builtin_amdgcn_sched_barrier(0);
        if (on) {
          const double x = solve_item<K, kGw, kOvf>(W, cur, c8, xv);
          if (kOne || cur.own) put(cur.at, x);
        }
        on = on_next;
        // between two levels of at most 64 items only the first wave works, and
        // it waits for nobody
        const bool wide_next = !kOneWave && (pe - pb) * gw > 64;
        if (wide || wide_next)
          lds_barrier();  // LDS only: the global x is read only across a window restart
        else
          wave_lds_barrier();
        wide = wide_next;
        stamp(l0 + l);
      };
      int32_t l = 0;
      for (; l + 1 < nlc; l += 2) {
        step(l, a, b);
        step(l + 1, b, a);
      }
      if (l < nlc) step(l, a, b);
    }
  } else {
    for (int32_t l = 0; l < W.NL; ++l) {
      const int32_t pb = lv[l], items = (lv[l + 1] - pb) * gw;
      for (int32_t t = tid; t < items; t += WG) {
        const int32_t s = kOne ? t : t / gw;
        const uint32_t c8 = kOne ? 0u : 8u * (uint32_t)(t - s * gw);
        Item<K> it;
        load_item<K, kGw>(W, pb + s, c8, it);
        double xv[K > 0 ? K : 1];
        load_x<K, kGw>(it, c8, xv);
        put(it.at, solve_item<K, kGw, kOvf>(W, it, c8, xv));
      }
      lds_barrier();
      stamp(l);
    }
  }
}

// Phase 1: (row, rhs) items per thread whose loads are in flight together,
// and 16-byte image units per thread per copy round.
template <int WG, bool kOne>
constexpr int p1_items() {
  return WG >= 1024 ? (kOne ? 5 : 4) : WG >= 512 ? 6 : 8;
}
template <int WG>
constexpr int p1_copy() {
  return WG >= 1024 ? 8 : 12;
}

// Touches what phase 1 of window w reads (image, dependency ranges and lists,
// rows, right-hand sides), a cache line at a time, by threads t of nt: phase 1 is
// a chain of dependent reads, some 8 us for a small window straight from memory.
// Called by the waves that have no levels to solve meanwhile. Returns a value
// that depends on every read.
__device__ __forceinline__ unsigned touch_window(const int4 *__restrict__ win, int32_t w, int32_t gw, int32_t c0,
                                                 const ThinArgs &A, int t, int nt) {
  const int4 W = win[w];
  const int32_t P0 = A.level_ptr[W.x], P1 = A.level_ptr[win[w + 1].x], R = P1 - P0;
  const int32_t nu = (int32_t)window_image_units(R, W.z, (W.y >> 2) & 3);
  const uint4 *im = A.img + W.w;
  unsigned sink = 0;
  for (int32_t u = t * 8; u < nu; u += nt * 8) sink ^= im[u].x;
  for (int32_t u = t * 32; u <= R; u += nt * 32) sink ^= (unsigned)A.ext_ptr[P0 + u];
  const int32_t e0 = A.ext_ptr[P0], e1 = A.ext_ptr[P1];
  for (int32_t e = e0 + t * 8; e < e1; e += nt * 8) sink ^= (unsigned)A.ext[e].col;
  // rows of a level lie near one another: every eighth finds most lines of b
  for (int32_t i = t; i < (R + 7) / 8 * gw; i += nt) {
    const int32_t row = A.rio.perm[P0 + 8 * (i / gw)], c = c0 + i % gw;
    sink ^= (unsigned)__double_as_longlong(A.rio.b[(int64_t)row * A.rio.rs + (int64_t)c * A.rio.cs]);
  }
  return sink;
}

// How long a wave that waits sleeps between polls, in units of 64 cycles.
constexpr int kPollSleep = 1;

// One window, by the calling workgroup, for the ng right-hand sides c0 .. c0 +
// ng - 1 of the nrhs (kOne: ng = 1): the columns are independent, LDS holds ng
// values per row. Returns the latched error bits; a window that does not fit is
// an error.
// kSplit: ng < nrhs; without it the strides and the first column are
// compile-time where they can be.
// kPoll: earlier windows may still be in progress on other workgroups. Every
// unfinished x then reads as kPendingX, so a load of it returns "done" and the
// value at once: a row's sum takes the finished values first (they come first:
// ascending positions), then waits for the others past the caches. A wave that
// has not moved for tlimit ticks of the wall clock gives up (time-out); with
// whole_launch it does so tlimit ticks after t0, however it moved.
// rot: the first thread of the wave that solves the levels of at most 64 items.
// touch_next: the other waves bring the next window's data nearer meanwhile.
template <int WG, int kGw, int kTime, bool kSplit, bool kPoll>
__device__ __forceinline__ int solve_window(char *lds_raw, const int4 *__restrict__ win, int32_t w, int32_t nrhs,
                                            int32_t ng, int32_t c0_arg, const ThinArgs &A, const Times &T,
                                            unsigned long long t0, unsigned long long tlimit, bool whole_launch,
                                            int rot, bool touch_next) {
  constexpr bool kOne = kGw == 1;
  const int32_t nr = kOne && !kSplit ? 1 : nrhs;  // stride of the global vectors
  const int32_t gw = kGw > 0 ? kGw : ng;          // columns in LDS and per row of items
  const int32_t c0 = kSplit ? c0_arg : 0;         // the first of those columns
  const int tid = threadIdx.x;
  const int32_t *__restrict__ level_ptr = A.level_ptr;
  const int32_t *__restrict__ ext_ptr = A.ext_ptr;
  const ExtDep *__restrict__ ext = A.ext;
  const double *__restrict__ bp = A.bp;
  double *xp = A.xp;
  // where the x of earlier windows is read: the work vector by position, or the
  // caller's x by row
  const double *xs = A.rio.x ? A.rio.x : xp;
  auto at_x = [&](int32_t k, int32_t c) -> int64_t {
    return A.rio.x ? (int64_t)k * A.rio.rs + (int64_t)c * A.rio.cs : (int64_t)k * nr + c;
  };
  int bits = 0;
  unsigned long long t_w0 = 0, t_prev = 0;
  float p1_per_row = 0.f;
  if (kTime == kDurations && tid == 0) t_w0 = wall_clock64();
  const int4 W = win[w];
  const int32_t lA = W.x, lB = win[w + 1].x, flags = W.y;
  const int32_t P0 = level_ptr[lA], P1 = level_ptr[lB];
  const int32_t R = P1 - P0;
  const int32_t NO = W.z;  // the window's overflow records
  const int32_t NL = lB - lA;
  const int kc = (flags >> 2) & 3;
  // the host sizes windows to fit, and 16-bit slots and offsets must hold R and NO
  if (thin_window_bytes(R, NO, NL, gw, kc) > A.lds - kCtlBytes || R >= 65536 || NO >= 65536) return EB_ARG;
  Win X;
  X.rec = kCtlBytes + (uint32_t)window_x_bytes(R, gw);
  X.ovf = X.rec + 16 * (uint32_t)window_record_units(R, kc);
  int32_t *lv = reinterpret_cast<int32_t *>(lds_raw + X.ovf + 16 * NO);
  X.lv = lv;
  X.NL = NL, X.gw = gw;
  const int32_t nu = (int32_t)window_image_units(R, NO, kc);
  double *v = reinterpret_cast<double *>(lds_raw + kCtlBytes);
  // phase 1. Each thread requests its items' right-hand side and range of
  // dependencies before the window; in the first round it streams
  // the window's static image into LDS while those are in flight; then it
  // subtracts the dependencies before the window (in the row's order).
  const int32_t nitems = R * gw;
  constexpr int kI = p1_items<WG, kOne>();
  for (int32_t base = 0; base < nitems; base += WG * kI) {
    double acc[kI];
    int32_t e0[kI], e1[kI];
    // row and column of the thread's first item; the next is WG items on, which
    // kCol divides for a constant number of columns
    const int32_t sb = kOne ? base + tid : (base + tid) / gw;
    const int32_t cb = kOne ? 0 : base + tid - sb * gw;
    constexpr bool kCol = kGw > 0 && WG % (kGw > 0 ? kGw : 1) == 0;
    auto col_of = [&](int j) -> int32_t {
      if (kCol) return c0 + cb;
      const int32_t it = base + j * WG + tid;
      return c0 + it % gw;
    };
#pragma unroll
    for (int j = 0; j < kI; ++j) {
      const int32_t it = base + j * WG + tid;
      const int32_t sj = kCol ? (it < nitems ? sb + j * (WG / (kGw > 0 ? kGw : 1)) : R - 1)
                              : (it < nitems ? it : nitems - 1) / gw;
      const int32_t pos = P0 + sj;
      const int32_t cj = col_of(j);
      // right-hand sides stored by rows: the caller's b through the level
      // order, except rows of T with off-diagonals (b' in bp)
      if (A.rio.b && !(A.rio.tflag && A.rio.tflag[pos]))
        acc[j] = A.rio.b[at_x(A.rio.perm[pos], cj)];
      else
        acc[j] = bp[(int64_t)pos * nr + cj];
      e0[j] = ext_ptr[pos];
      e1[j] = it < nitems ? ext_ptr[pos + 1] : e0[j];
    }
    if (base == 0) {
      for (int32_t i = tid; i <= NL + 1; i += WG) lv[i] = level_ptr[lA + (i <= NL ? i : NL)] - P0;
      for (int32_t i = tid; i < gw; i += WG) v[(int64_t)R * gw + i] = 0.0;
      const uint4 *__restrict__ im = A.img + W.w;
      uint4 *dst = reinterpret_cast<uint4 *>(lds_raw + X.rec);
      constexpr int kC = p1_copy<WG>();
      for (int32_t u0 = 0; u0 < nu; u0 += WG * kC) {
        uint4 t[kC];
#pragma unroll
        for (int j = 0; j < kC; ++j) {
          const int32_t u = u0 + j * WG + tid;
          t[j] = im[u < nu ? u : nu - 1];
        }
#pragma unroll
        for (int j = 0; j < kC; ++j) {
          const int32_t u = u0 + j * WG + tid;
          if (u < nu) dst[u] = t[j];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kI; ++j) {
      const int32_t it = base + j * WG + tid;
      if (it >= nitems) continue;
      const int32_t c = col_of(j);
      double a = acc[j];
      int32_t e = e0[j];
      while (e < e1[j]) {
        double wv[kBatch], xv[kBatch];
        int32_t k[kBatch];
        const int32_t cnt = e1[j] - e < kBatch ? e1[j] - e : kBatch;
#pragma unroll
        for (int d = 0; d < kBatch; ++d) {
          const ExtDep x = ext[e + (d < cnt ? d : 0)];
          wv[d] = x.w;
          k[d] = A.rio.x ? x.row : x.col;
        }
        // by rows the caller's x is the work vector, read by caller row
#pragma unroll
        for (int d = 0; d < kBatch; ++d) xv[d] = xs[at_x(k[d], c)];
        int32_t done = 0;
#pragma unroll
        for (int d = 0; d < kBatch; ++d) {
          if (d < cnt && (!kPoll || (done == d && !is_pending(xv[d])))) {
            a = fma(-wv[d], xv[d], a);
            done = d + 1;
          }
        }
        e += done;
        if (kPoll && done < cnt) break;
      }
      acc[j] = a;
      e0[j] = e;
      v[(int64_t)it] = a;
    }
    if constexpr (kPoll) {
      // what is left is polled past the caches, all items of a thread at once:
      // the next two dependencies of each are requested together, and the
      // finished ones taken in order
      constexpr int kP = 2;
      unsigned spins = 0;
      int32_t rest0 = -1;  // dependencies left at the last look at the clock
      WaitLimit wait{t0, false};
      for (;;) {
        bool left[kI], any = false, moved = false;
        double wv[kI][kP];
        unsigned long long xv[kI][kP];
#pragma unroll
        for (int j = 0; j < kI; ++j) {
          left[j] = __ballot(e0[j] < e1[j]) != 0ull;  // uniform over the wave
          any = any || left[j];
        }
        if (!any) break;
#pragma unroll
        for (int j = 0; j < kI; ++j) {
          if (!left[j]) continue;
          const int32_t c = col_of(j);
#pragma unroll
          for (int d = 0; d < kP; ++d) {
            const ExtDep x = ext[e0[j] + d < e1[j] ? e0[j] + d : e1[j] > 0 ? e1[j] - 1 : 0];
            wv[j][d] = x.w;
            xv[j][d] = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(xs) +
                                             at_x(A.rio.x ? x.row : x.col, c),
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
#pragma unroll
        for (int j = 0; j < kI; ++j) {
          if (!left[j]) continue;
          const int32_t left_j = e1[j] - e0[j];
          int32_t done = 0;
#pragma unroll
          for (int d = 0; d < kP; ++d) {
            if (d < left_j && done == d && xv[j][d] != kPendingX) {
              acc[j] = fma(-wv[j][d], __longlong_as_double((long long)xv[j][d]), acc[j]);
              done = d + 1;
            }
          }
          e0[j] += done;
          moved = moved || done > 0;
          if (done > 0 && e0[j] == e1[j]) v[(int64_t)(base + j * WG + tid)] = acc[j];
        }
        if (__ballot(moved) == 0ull) __builtin_amdgcn_s_sleep(kPollSleep);
        if ((++spins & 63u) == 0u) {
          int32_t rest = 0;
#pragma unroll
          for (int j = 0; j < kI; ++j) rest += e1[j] - e0[j];
          wait.moved = !whole_launch && __ballot(rest != rest0) != 0ull;
          rest0 = rest;
          if (wait.expired(wall_clock64(), tlimit)) {
            bits |= EB_TIMEOUT;
            break;
          }
        }
      }
    }
  }
  __syncthreads();
  if (kTime == kDurations && tid == 0) {
    t_prev = wall_clock64();
    p1_per_row = R > 0 ? (float)(t_prev - t_w0) * T.ns_per_tick / (float)R : 0.f;
  }
  // x goes to global memory as it is solved where a window's place there is a
  // fixed multiple of its place in LDS (all columns, or one of them), except
  // from a lone wave, whose every instruction lengthens a level (20 ns a level,
  // more than the 0.3 us a window's x arrives earlier): the other waves store
  // its x at the end of the window
  const bool now = kPoll && !(flags & 1) && !A.rio.x && (kOne || gw == nr);
  double *gx = xp + (int64_t)P0 * nr + c0;
  const uint32_t gmul = kSplit ? (uint32_t)nr : 1u;
  const int vt = (tid + WG - rot) & (WG - 1);
  unsigned sink = 0;
  if (touch_next && vt >= 64) sink = touch_window(win, w + 1, gw, c0, A, vt - 64, WG - 64);
#define LEVELS(K, OVF)                                                                                             \
  if (flags & 1) {                                                                                                 \
    if (vt < 64)                                                                                                   \
      solve_levels<WG, kGw, K, OVF, true, kTime, false>(X, flags, lA, T, t_prev, p1_per_row, gx, gmul, vt);       \
  } else if (kPoll && now) {                                                                                       \
    solve_levels<WG, kGw, K, OVF, false, kTime, kPoll>(X, flags, lA, T, t_prev, p1_per_row, gx, gmul, vt);        \
  } else {                                                                                                         \
    solve_levels<WG, kGw, K, OVF, false, kTime, false>(X, flags, lA, T, t_prev, p1_per_row, gx, gmul, vt);        \
  }
  if (kc == 0 && NO == 0) {
    LEVELS(2, false)
  } else if (kc == 0) {
    LEVELS(2, true)
  } else if (kc == 1 && NO == 0) {
    LEVELS(6, false)
  } else if (kc == 1) {
    LEVELS(6, true)
  } else if (kc == 2) {
    LEVELS(10, true)
  } else {
    LEVELS(0, false)
  }
#undef LEVELS
  if (sink == 0x9e3779b9u) A.tp[1] = sink;  // keeps the reads; the word is never read
  __syncthreads();  // every x of the window is in LDS
  for (int32_t i = tid; i < nitems; i += WG) {
    const double x = v[i];
    if (!isfinite(x)) bits |= EB_NONFINITE;
    if (now) continue;
    const int32_t sj = kOne ? i : i / gw;
    const int32_t cj = c0 + (kOne ? 0 : i - sj * gw);
    // by rows: the caller's x only
    double *to = A.rio.x ? A.rio.x + at_x(A.rio.perm[P0 + sj], cj)
                 : gw == nr ? xp + (int64_t)P0 * nr + i
                            : xp + (int64_t)(P0 + sj) * nr + cj;
    if (kPoll)
      put_x(to, x);
    else
      *to = x;
  }
  __syncthreads();  // the window's global x is complete before the next phase 1 of this workgroup reads it
  return bits;
}

// The windows [win, win + nwin) of one thin run one after another, by the
// calling workgroup.
template <int WG, int kGw, int kTime, bool kSplit = false>
__device__ __forceinline__ int thin_run_body(char *lds_raw, const int4 *__restrict__ win, int32_t nwin, int32_t nrhs,
                                             int32_t ng, int32_t c0, const ThinArgs &A, const Times &T, int rot = 0,
                                             bool touch = false) {
  int bits = 0;
  for (int32_t w = 0; w < nwin && !(bits & EB_ARG); ++w)
    bits |= solve_window<WG, kGw, kTime, kSplit, false>(lds_raw, win, w, nrhs, ng, c0, A, T, 0, 0, false, rot,
                                                        touch && w + 1 < nwin);
  return bits;
}

// First column of group g of ng columns. Where ng does not divide nrhs the last
// group overlaps the one before: both write the same values to its columns.
__device__ __forceinline__ int32_t first_col(int32_t g, int32_t nrhs, int32_t ng) { return min(g * ng, nrhs - ng); }

// One thin run in one workgroup per group of ng columns. For runs of one window, and for the labelling
// runs that time levels.
template <int WG, bool kOne, int kTime = kNoTimes, bool kSplit = false>
__global__ __launch_bounds__(WG) void k_thin_run(const int4 *__restrict__ win, int32_t nwin, int32_t nrhs, int32_t ng,
                                                 ThinArgs A, int *err, Times T) {
  extern __shared__ __align__(16) char lds_raw[];
  const int bits = thin_run_body<WG, kOne ? 1 : 0, kTime, kSplit>(
      lds_raw, win, nwin, nrhs, ng, first_col((int32_t)blockIdx.x, nrhs, ng), A, T);
  if (bits) atomicOr(err, bits);
}

// One thin run with its windows spread over workgroups. A single workgroup
// spends a window's phase 1 (about 100 KB of records, b' and dependencies
// through one CU's memory pipeline: 4 to 6 us for 3,000 rows) and the store of
// its x between the levels of one window and of the next; here the windows
// after the one being solved are loaded by other workgroups meanwhile, and each
// waits only for the x it reads (solve_window, kPoll), so what is left of a
// window is its levels and one hand-over, about 0.5 us.
// Windows are taken in order from a ticket counter, so the ones a window waits
// for belong to running workgroups and every wait ends. Columns are
// independent: group g of ng columns is a chain of its own. Lane l of nlane
// holds groups l, l + nlane, ... on the workgroups with blockIdx mod 8 = l, those
// of one XCD (workgroups are dealt to the 8 XCDs in turn), where a hand-over
// takes 425 ns instead of 558 and the windows share an L2 (64 workgroups on all
// XCDs took the same time on the power law). tp[kTicketStride * (1 + l)] is
// lane l's ticket counter, tp[0] counts the workgroups that are done, and the
// last one clears both.
// Measured, one right-hand side: the rewritten 2D stencil 1000^2 + chain 1.44 ms a
// solve against 2.69 with one workgroup (and four that prefetched into its L2),
// the 300^2 one with its 4,001-row tail 0.74 against 0.89.
constexpr int kXcd = 8;
template <int WG, bool kOne, bool kSplit, int kTime = kNoTimes>
__global__ __launch_bounds__(WG) void k_thin_pipe(const int4 *__restrict__ win, int32_t nwin, int32_t nrhs, int32_t ng,
                                                  int32_t nlane, ThinArgs A, int *err, unsigned long long tlimit,
                                                  int whole_launch, Times T) {
  extern __shared__ __align__(16) char lds_raw[];
  const int32_t lane = (int32_t)blockIdx.x % kXcd;
  if (lane >= nlane) return;
  int32_t &s_t = reinterpret_cast<Ctl *>(lds_raw)->next;
  const int32_t groups = (nrhs + ng - 1) / ng;
  const int32_t mine = (groups - lane + nlane - 1) / nlane;  // groups of this lane
  unsigned *ticket = A.tp + kTicketStride * (1 + lane);
  const unsigned long long t0 = wall_clock64();
  int bits = 0;
  while (!(bits & EB_ARG)) {
    if (threadIdx.x == 0)
      s_t = (int32_t)__hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int32_t t = s_t;
    __syncthreads();
    if (t >= nwin * mine) break;
    const int32_t w = t / mine, g = lane + nlane * (t - w * mine);
    bits |= solve_window<WG, kOne ? 1 : 0, kTime, kSplit, true>(lds_raw, win, w, nrhs, ng, first_col(g, nrhs, ng), A, T,
                                                                t0, tlimit, whole_launch != 0, 0, false);
  }
  if (bits) atomicOr(err, bits);
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned active = gridDim.x / kXcd * (unsigned)nlane;
    if (__hip_atomic_fetch_add(A.tp, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == active - 1) {
      for (int32_t l = 0; l < nlane; ++l) atomicExch(A.tp + kTicketStride * (1 + l), 0u);
      atomicExch(A.tp, 0u);
    }
  }
}

// Marks the x of positions [p0, p0 + rows) as unfinished; by rows through perm.
__global__ void k_fill_pending(int64_t p0, int64_t rows, int32_t nr, const int32_t *__restrict__ perm, double *x) {
  unsigned long long *xb = reinterpret_cast<unsigned long long *>(x);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < rows * nr; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / nr;
    xb[perm ? (int64_t)perm[p0 + r] * nr + (i - r * nr) : p0 * nr + i] = kPendingX;
  }
}

// A row's first four off-diagonals (column position, value), -1 / 0 padded.
__global__ void k_fill_ell(int32_t n, const int32_t *__restrict__ srp, const int32_t *__restrict__ sci,
                           const double *__restrict__ sva, int4 *ell_c, double2 *ell_v) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
    const int32_t qb = srp[p], deg = srp[p + 1] - qb;
    int32_t c[4];
    double v[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      c[d] = d < deg ? sci[qb + d] : -1;
      v[d] = d < deg ? sva[qb + d] : 0.0;
    }
    ell_c[p] = make_int4(c[0], c[1], c[2], c[3]);
    ell_v[2 * p] = make_double2(v[0], v[1]);
    ell_v[2 * p + 1] = make_double2(v[2], v[3]);
  }
}

// Many independent matrices in one persistent launch: each workgroup takes
// the next task, a group of ng columns of a matrix, from a device queue
// (matrices are queued deepest first) and solves it window by window; b and x
// are read and written in the caller's layout. The last workgroup to finish
// resets the queue, so the launch can be replayed (graph capture) without a
// host-side reset. q[0] = next ticket, q[1] = finished workgroups.
// A task is a chain of levels, so what counts is how many chains are under way:
// groups of a few columns (the host chooses), and as many workgroups per CU as
// registers and LDS allow (1 of 1,024 threads, 2 of 512, 4 of 256). Workgroups fill the CUs one after another, so those of a CU
// are `cus` apart; each has another of its first four waves, which sit on the
// four SIMDs, solve its narrow levels. Waves without levels touch the next
// window's data meanwhile. The vectors pass through HBM once each way instead of
// three times (copied to level order and back, 2.36 ms of 5.6 on the workload
// below). Bound by the levels and by phase 1 of the windows, some 10 us of
// dependent reads each: 512 matrices of 1,000 to 50,000 rows, 16 columns, 3.9 ms
// against 6.6 with all columns of a matrix in one workgroup.
template <int WG, int kGw>
__global__ __launch_bounds__(WG, 4) void k_batch_run(int32_t nmat, const int32_t *__restrict__ order,
                                                     const int32_t *__restrict__ mwin, const int4 *__restrict__ win,
                                                     int32_t nrhs, int32_t ng, const int64_t *__restrict__ row_off,
                                                     ThinArgs A, unsigned *q, int *err, int cus) {
  extern __shared__ __align__(16) char lds_raw[];
  int32_t &s_m = reinterpret_cast<Ctl *>(lds_raw)->next;
  const int32_t groups = (nrhs + ng - 1) / ng;
  const double *b0 = A.rio.b;
  double *x0 = A.rio.x;
  int bits = 0;
  const int rot = 64 * (int)(blockIdx.x / (unsigned)cus % 4u);
  for (;;) {
    if (threadIdx.x == 0) s_m = (int32_t)atomicAdd(q, 1u);
    __syncthreads();
    const int32_t t = s_m;
    __syncthreads();
    if (t >= nmat * groups) break;
    const int32_t i = t / groups, m = order[i];
    // entry (r, c) of matrix m is at nrhs * off + c * n + (r - off)
    const int64_t off = row_off[m], n = row_off[m + 1] - off;
    A.rio.b = b0 + (nrhs - 1) * off;
    A.rio.x = x0 + (nrhs - 1) * off;
    A.rio.rs = 1;
    A.rio.cs = n;
    bits |= thin_run_body<WG, kGw, kNoTimes, true>(lds_raw, win + mwin[m], mwin[m + 1] - mwin[m] - 1, nrhs, ng,
                                                   first_col(t - i * groups, nrhs, ng), A, Times{}, rot, true);
  }
  if (threadIdx.x == 0) {
    if (bits) atomicOr(err, bits);
    __threadfence();
    if (atomicAdd(q + 1, 1u) == gridDim.x - 1) {
      q[0] = 0;
      q[1] = 0;
      __threadfence();
    }
  }
}

template <int WG, bool kOne>
void set_lds_attr() {
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_thin_pipe<WG, kOne, false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kWinBytes);
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_thin_pipe<WG, kOne, true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kWinBytes);
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_thin_run<WG, kOne>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kWinBytes);
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_thin_run<WG, kOne, kNoTimes, true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kWinBytes);
}

// Workgroups that hold windows of one chain of a spread thin run (6, 12 and 24
// took the same time on the 2D stencils).
constexpr int kPipeDepth = 8;

}  // namespace

bool thin_piped(int32_t nwin, unsigned long long tlimit) { return nwin >= 2 && tlimit > 0; }

int thin_win_bytes() { return kWinBytes - kCtlBytes; }
int thin_ctl_bytes() { return kCtlBytes; }

namespace {
template <int WG>
void batch_attr() {
  const void *f[] = {reinterpret_cast<const void *>(&k_batch_run<WG, 0>),
                     reinterpret_cast<const void *>(&k_batch_run<WG, 1>),
                     reinterpret_cast<const void *>(&k_batch_run<WG, 4>)};
  for (const void *k : f) (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kWinBytes);
}
}  // namespace

void solve_kernels_init() {
  set_lds_attr<256, true>();
  set_lds_attr<256, false>();
  set_lds_attr<512, true>();
  set_lds_attr<512, false>();
  set_lds_attr<1024, true>();
  set_lds_attr<1024, false>();
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_thin_run<512, true, kDurations>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kWinBytes);
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_thin_run<512, false, kDurations>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kWinBytes);
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_thin_pipe<1024, true, true, kFinish>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kWinBytes);
  batch_attr<256>();
  batch_attr<512>();
  batch_attr<1024>();
}

hipError_t launch_fill_pending(int64_t p0, int64_t rows, int32_t nr, const int32_t *perm, double *x, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_pending, dim3(grid_for(rows * nr, 256, 4096)), dim3(256), 0, s, p0, rows, nr, perm, x);
  return hipGetLastError();
}

namespace {
// A spread run: lanes (XCDs) and workgroups. kPipeDepth workgroups per chain on
// the chain's XCD; not more than hold windows, nor more than its CUs (a workgroup
// takes a CU's LDS).
struct PipeGrid {
  int32_t nlane;
  unsigned blocks;
};
PipeGrid pipe_grid(int32_t nwin, int32_t groups) {
  const int32_t nlane = groups < kXcd ? groups : kXcd;
  const int32_t chains = (groups + nlane - 1) / nlane;
  const int64_t depth = std::min<int64_t>({(int64_t)kPipeDepth * chains, (int64_t)nwin * chains, 32});
  return PipeGrid{nlane, (unsigned)depth * kXcd};
}
}  // namespace

hipError_t launch_thin_stamped(const int4 *win, int32_t nwin, int32_t nrhs, const ThinArgs &a, int *err, hipStream_t s,
                               unsigned long long *finish, int32_t nlev, unsigned long long tlimit) {
  const PipeGrid g = pipe_grid(nwin, nrhs);
  hipLaunchKernelGGL((k_thin_pipe<1024, true, true, kFinish>), dim3(g.blocks), dim3(1024), kWinBytes, s, win, nwin,
                     nrhs, 1, g.nlane, a, err, tlimit, 1, Times{nullptr, 0.f, finish, nlev});
  return hipGetLastError();
}

hipError_t launch_thin_run(int wg, const int4 *win, int32_t nwin, int32_t nrhs, const ThinArgs &a, int *err,
                           hipStream_t s, float *times, float ns_per_tick, int32_t ng, unsigned long long tlimit,
                           bool whole_launch) {
  if (ng <= 0 || ng > nrhs || times) ng = nrhs;  // labelling runs are never split
  const bool one = ng == 1;
  const bool split = ng < nrhs;
  const int32_t groups = (nrhs + ng - 1) / ng;
  if (times) {  // labelling runs only: 512 threads
    const Times T{times, ns_per_tick, nullptr, 0};
    if (one)
      hipLaunchKernelGGL((k_thin_run<512, true, kDurations>), dim3(1), dim3(512), kWinBytes, s, win, nwin, nrhs, ng, a,
                         err, T);
    else
      hipLaunchKernelGGL((k_thin_run<512, false, kDurations>), dim3(1), dim3(512), kWinBytes, s, win, nwin, nrhs, ng,
                         a, err, T);
    return hipGetLastError();
  }
  const bool pipe = thin_piped(nwin, tlimit);
  const PipeGrid g = pipe_grid(nwin, groups);
#define THIN(W, ONE, SPLIT)                                                                                       \
  if (pipe)                                                                                                       \
    hipLaunchKernelGGL((k_thin_pipe<W, ONE, SPLIT>), dim3(g.blocks), dim3(W), kWinBytes, s, win, nwin, nrhs, ng,   \
                       g.nlane, a, err, tlimit, whole_launch ? 1 : 0, Times{});                                   \
  else                                                                                                            \
    hipLaunchKernelGGL((k_thin_run<W, ONE, kNoTimes, SPLIT>), dim3((unsigned)groups), dim3(W), kWinBytes, s, win,  \
                       nwin, nrhs, ng, a, err, Times{});
#define THINW(W)              \
  if (split && one) {         \
    THIN(W, true, true)       \
  } else if (split) {         \
    THIN(W, false, true)      \
  } else if (one) {           \
    THIN(W, true, false)      \
  } else {                    \
    THIN(W, false, false)     \
  }
  if (wg == 256) {
    THINW(256)
  } else if (wg == 1024) {
    THINW(1024)
  } else {
    THINW(512)
  }
#undef THINW
#undef THIN
  return hipGetLastError();
}

hipError_t launch_fill_ell(int32_t n, const int32_t *srp, const int32_t *sci, const double *sva, int4 *ell_c,
                           double2 *ell_v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_ell, dim3(grid_for(n, 256, 16384)), dim3(256), 0, s, n, srp, sci, sva, ell_c, ell_v);
  return hipGetLastError();
}

int batch_lds(int wg) { return wg == 256 ? 39 * 1024 : wg == 512 ? 79 * 1024 : kWinBytes; }

hipError_t launch_batch_run(int wg, int32_t nmat, int32_t grid, const int32_t *order, const int32_t *mwin,
                            const int4 *win, int32_t nrhs, int32_t ncol, const int64_t *row_off, const ThinArgs &a,
                            unsigned *q, int *err, hipStream_t s) {
  int dev = 0, cus = 256;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  cus = std::max(cus, 1);
#define BATCHG(W, G)                                                                                            \
  hipLaunchKernelGGL((k_batch_run<W, G>), dim3(grid), dim3(W), a.lds, s, nmat, order, mwin, win, nrhs, ncol, \
                     row_off, a, q, err, cus);
#define BATCH(W)          \
  if (ncol == 1) {        \
    BATCHG(W, 1)          \
  } else if (ncol == 4) { \
    BATCHG(W, 4)          \
  } else {                \
    BATCHG(W, 0)          \
  }
  if (wg == 256) {
    BATCH(256)
  } else if (wg == 1024) {
    BATCH(1024)
  } else {
    BATCH(512)
  }
#undef BATCH
#undef BATCHG
  return hipGetLastError();
}

int batch_resident_blocks(int wg, int lds) {
  int dev = 0, cus = 256, occ = 1;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const void *f = wg == 256    ? reinterpret_cast<const void *>(&k_batch_run<256, 0>)
                  : wg == 1024 ? reinterpret_cast<const void *>(&k_batch_run<1024, 0>)
                               : reinterpret_cast<const void *>(&k_batch_run<512, 0>);
  (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, f, wg, lds);
  return cus * (occ > 0 ? occ : 1);
}
