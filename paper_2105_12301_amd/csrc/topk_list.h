// Register top-k lists of (float32 key, index) entries, shared by the exact
// scans, the filtered scan and the subsample scan.
//
// An entry is one 64-bit word with the key's bits above the index, held as a
// double: keys are sums of squares (never negative, never -0), so their bit
// patterns, and with them the words read as doubles, order exactly as
// (key, index) lexicographically, ties to the lower index included.  (The
// high word of a finite key, of +inf and of the default NaN stays below the
// double exponent 0x7ff, and float64 minimum and maximum keep subnormal words
// bit for bit.)  v_min_f64 / v_max_f64 issue in 4.7 cycles per wave on gfx950,
// like a single compare, conditional move or float32 median, so a sorted
// insertion costs two instructions a slot where separate key and index arrays
// take four (compare, two moves, median), and a compare-exchange two where
// they take seven.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace edm {

__device__ __forceinline__ double entry_min(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double entry_max(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double entry(float key, int q) { return __hiloint2double(__float_as_int(key), q); }
__device__ __forceinline__ float entry_key(double e) { return __int_as_float(__double2hiint(e)); }
__device__ __forceinline__ int entry_idx(double e) { return __double2loint(e); }
// An empty slot: after every finite key.  A candidate whose key is +inf (or
// NaN) is never below it, so it is never listed.
__device__ __forceinline__ double entry_empty() { return entry(__builtin_inff(), 0); }
// A slot of an idle list: before every candidate, so nothing enters.
__device__ __forceinline__ double entry_idle() { return entry(-1.0f, -1); }

// Sorted insertion of x into the slice [OFF, OFF + K).  An entry not below the
// last one (an empty entry always) leaves the slice unchanged, so a whole wave
// runs it without lane masking.
template <int OFF, int K, int TOT>
__device__ __forceinline__ void list_insert(double (&l)[TOT], double x) {
#pragma unroll
  for (int i = K - 1; i > 0; --i) l[OFF + i] = entry_min(l[OFF + i], entry_max(l[OFF + i - 1], x));
  l[OFF] = entry_min(l[OFF], x);
}

// l[OFF, OFF + K) := the K smallest entries of itself and of a second sorted
// list other(0 .. K-1), sorted.  [own ascending, maxima, other descending] is
// bitonic; its first half-cleaner stage (elementwise minimum) leaves the N
// smallest as a bitonic sequence and the remaining stages sort it.  Blocks
// that start at or beyond K only order entries that are dropped.
template <int OFF, int K, int TOT, class F>
__device__ __forceinline__ void list_merge(double (&l)[TOT], F &&other) {
  constexpr int N = K <= 1 ? 1 : (K <= 2 ? 2 : (K <= 4 ? 4 : (K <= 8 ? 8 : (K <= 16 ? 16 : 32))));
  static_assert(K <= 32 && (N == 1 || N - K < K), "every position of the lower half holds an entry");
  double c[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int j = N - 1 - i;  // the other list's entry facing position i, if j < K
    if (i < K && j < K) c[i] = entry_min(l[OFF + i], other(j));
    else c[i] = i < K ? l[OFF + i] : other(j);
  }
#pragma unroll
  for (int d = N / 2; d > 0; d >>= 1)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if ((i & d) == 0 && (i & ~(2 * d - 1)) < K) {
        const double a0 = c[i], a1 = c[i + d];
        c[i] = entry_min(a0, a1);
        c[i + d] = entry_max(a0, a1);
      }
#pragma unroll
  for (int i = 0; i < K; ++i) l[OFF + i] = c[i];
}

// Pending insertions of an exact scan.  A wave's lanes improve their lists at
// different candidates, so inserting as they come runs the whole insertion on
// nearly every step of a wave (the union over 64 lanes).  Instead a lane
// queues its improving entries in LDS (one row of 64 entries per queue
// position, so a wave's accesses are contiguous), and when some lane may run
// out of room the wave inserts them position by position: as many insertions
// as the fullest lane holds, not as many as the union of steps.  The k-th key
// a lane tests against is the one of the last flush, so entries that no longer
// enter are queued too; the insertion leaves the list as it is for them.
// (Where this pays: queue_wins below.)
constexpr int kPend = 8;          // queue positions per lane
constexpr int kPendStep = 4;      // candidates between two looks at the fill
constexpr int kPendBytes = kPend * 8 * 64;  // LDS per wave

// (The branch around the write is the better form where scans are long and
// improving entries rare: writing every entry and moving the end of the queue
// only where wanted took 694 against 572 ms for 20 scans of 10000 x 2000.)
struct Pending {
  double *at;  // this lane's entry of position 0
  int n = 0;
  __device__ __forceinline__ explicit Pending(double *area)
      : at(area + (threadIdx.x / 64) * (kPend * 64) + (threadIdx.x & 63)) {}
  __device__ __forceinline__ void push(double e, bool want) {
    if (want) {
      at[n * 64] = e;
      ++n;
    }
  }
  // (wave-uniform) some lane may lack room for another kPendStep entries
  __device__ __forceinline__ bool full() const {
    return __builtin_amdgcn_ballot_w64(n > kPend - kPendStep) != 0;
  }
  template <class F>
  __device__ __forceinline__ void drain(F &&insert) {
#pragma unroll 1
    for (int i = 0; i < kPend; ++i) {
      const bool has = i < n;
      if (__builtin_amdgcn_ballot_w64(has) == 0) break;
      const double e = at[i * 64];
      insert(has ? e : entry_empty());
    }
    n = 0;
  }
};

// Layouts of an exact scan's workgroup: Q waves of 64 queries, each query's
// candidates split over S waves (workgroup = 64 Q S threads), improving
// candidates inserted from a queue or as they come (scan_layout).
// Merge of the S lists of every query into the lists of split 0: in each
// round the upper half of the splits left writes its lists to LDS.
// (k_knn's epilogue takes the area over: 12 bytes an entry and query, which
// S / 2 lists of 8 bytes hold from S = 4 on.)
// area: merge_bytes<Q, S>(K) bytes; l: the lane's slice [OFF, OFF + K).
template <int Q, int S>
constexpr int merge_bytes(int K) {
  return S > 1 ? Q * (S / 2) * K * 64 * 8 : 0;
}
template <int Q, int S, int OFF, int K, int TOT>
__device__ __forceinline__ void merge_splits(double (&l)[TOT], double *area) {
  const int wave = static_cast<int>(threadIdx.x) / 64, lane = static_cast<int>(threadIdx.x) & 63;
  const int qg = wave % Q, sp = wave / Q;
#pragma unroll
  for (int half = S / 2; half > 0; half /= 2) {
    double *at = area + (static_cast<int64_t>(sp % half) * Q + qg) * (K * 64) + lane;
    __syncthreads();  // the area's previous use is over
    if (sp >= half && sp < 2 * half) {
#pragma unroll
      for (int i = 0; i < K; ++i) at[i * 64] = l[OFF + i];
    }
    __syncthreads();
    if (sp < half) list_merge<OFF, K, TOT>(l, [&](int j) { return at[j * 64]; });
  }
}

// LDS bytes of a scan: the staged series (lds_x floats), then the queues,
// whose space the merge takes over.
constexpr int64_t kLdsBytes = 160 * 1024, kLdsGrain = 1280;  // of a compute unit, and the steps it is given out in
constexpr int64_t kScanLdsMax = kLdsBytes - 4608;            // less the kernels' static LDS
template <int Q, int S>
constexpr int64_t scan_lds(int K, int64_t lds_x, bool queue) {
  const int64_t pend = queue ? static_cast<int64_t>(Q) * S * kPendBytes : 0;
  const int64_t merge = merge_bytes<Q, S>(K);
  return lds_x * 4 + (pend > merge ? pend : merge);
}

constexpr int kCus = 256;  // compute units of the chip

// Waves of a scan without splits that a compute unit holds: workgroups of Q
// waves with `lds` bytes each, where the registers leave room for `cap` waves
// and the launch has `blocks` blocks of 256 queries.
constexpr int64_t resident_waves(int Q, int64_t lds, int cap, int64_t blocks) {
  const int64_t fit = kLdsBytes / ((lds + kLdsGrain - 1) / kLdsGrain * kLdsGrain);
  const int64_t by_lds = fit * Q, by_regs = cap / Q * Q, by_work = (blocks * 4 + kCus - 1) / kCus;
  const int64_t w = by_lds < by_regs ? by_lds : by_regs;
  return w < by_work ? w : by_work;
}
// The staged series is shared by a workgroup, so a long one leaves the more
// waves in flight the larger the workgroup is: of 4, 8 and 16 waves (`most`)
// the smallest with the most resident waves; 0 where nothing fits.  lds(Q):
// all of a workgroup's LDS.  (One scan, E = 8, without queues: 100 series of
// 20000 25.6 ms by 4 waves, 17.8 by 8; 300 of 12000 at E = 16, whose registers
// hold 12 waves, 37.0 by 4, 45.5 by 8.)
template <class F>
constexpr int most_resident(int most, int cap, int64_t blocks, F &&lds) {
  int best = 0;
  int64_t waves = 0;
  for (int q = 4; q <= most; q *= 2) {
    const int64_t w = lds(q) <= kLdsBytes ? resident_waves(q, lds(q), cap, blocks) : 0;
    if (w > waves) {
      waves = w;
      best = q;
    }
  }
  return best;
}

// Queue or insertion as candidates come, in a scan of one E: an insertion
// costs 2 (E + 1) float64 instructions on nearly every step of a wave, a queue
// its pushes and 4 KB of LDS a wave, which long series need for waves in
// flight.  Measured, queue against none: E = 6 490 / 500 us (1000 x 1000), 3411
// / 3323 (2000 x 2000); E = 8 4405 / 4438 (2000 x 2000), 6299 / 5889 (512 x 5000);
// E = 12 8610 / 8784 (512 x 5000), 11669 / 10766 (256 x 8000); E = 20 17758 / 17907
// (256 x 8000), 54475 / 45873 (300 x 12000); E = 1 330 / 252 (1000 x 1000).
constexpr int kQueueE = 5;  // from here on
constexpr bool queue_wins(int E, int64_t L_max) { return E >= kQueueE && L_max <= 640 * (E - 4); }

// Registers of a scan of one E, in waves a compute unit holds (k_knn: 64 up to
// E = 6, 80 up to 9, 96 up to 11, 128 up to 16, 155 at 20).
constexpr int scan_wave_cap(int E) { return E <= 6 ? 32 : E <= 9 ? 24 : E <= 11 ? 20 : E <= 16 ? 16 : 12; }

enum class ScanLayout { kPlainQueue, kPlain, kLong8, kLong16, kSplit, kTableSplit };
constexpr int64_t kTableSplitGroups = kCus;

// Blocks of 256 queries up to which four waves share a query's candidates:
// two workgroups of 16 waves a CU while the lists are short; with long ones
// the merges cost more than the second round wins (384 blocks: E = 8 1000 samples
// 121 against 129 us unsplit, E = 12 173 / 168, 4000 samples 474 / 502; E = 16
// 225 / 206, 300 samples 114 / 103; E = 20 174 / 124; 256 blocks: faster at every E
// and length, E = 20 163 / 223).
constexpr int64_t split_blocks(int E, int64_t L_max) {
  return E <= 10 || (E <= 14 && L_max >= 2000) ? 2 * kCus : kCus;
}

// Layout of a launch over nslots series of up to L_max samples at dimension E
// with lists of K entries (wants_mom: the launch writes a sweep's co-moments).
// kTableSplit, kSplit: few workgroups.  A scan of m candidates is a chain of m
//   steps however many compute units are idle; splitting it over waves and
//   merging their lists (list_merge, log2 S rounds through LDS) shortens it.
//   kTableSplit writes tables only: a sweep's co-moments are merged per 256
//   queries.  Up to one group of 64 queries a CU, where it wins at every E and
//   length (one table of 10000 samples, E = 1, 12: 64, 173 us by 16 waves, 210, 525
//   by 4; 256 groups of 1000-sample series, E = 12: 42, 91); a second round
//   still wins (512 groups 76 / 94), a fourth loses (1024 140 / 96).
inline ScanLayout scan_layout(int64_t nslots, int64_t L_max, int E, int K, bool wants_mom) {
  const int64_t lds_x = L_max + 138;  // (scan_floats)
  const int64_t groups = (L_max + 63) / 64 * nslots, blocks = (L_max + 255) / 256 * nslots;
  const bool queue = E >= kQueueE;
  if (!wants_mom && groups <= kTableSplitGroups && scan_lds<1, 16>(K, lds_x, queue) <= kScanLdsMax)
    return ScanLayout::kTableSplit;
  if (blocks <= split_blocks(E, L_max) && scan_lds<4, 4>(K, lds_x, queue) <= kScanLdsMax) return ScanLayout::kSplit;
  if (queue_wins(E, L_max)) return ScanLayout::kPlainQueue;
  const int q = most_resident(E <= 4 ? 16 : 8, scan_wave_cap(E), blocks,
                              [&](int w) { return lds_x * 4 + 48 * w; });  // (48: a wave's co-moments)
  return q == 16 ? ScanLayout::kLong16 : q == 8 ? ScanLayout::kLong8 : ScanLayout::kPlain;
}

}  // namespace edm
