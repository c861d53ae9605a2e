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
// candidates split over S waves (workgroup = 64 Q S threads).
// (4, 1): the plain layout.
// (16, 1), then (8, 1): long series, whose staged samples leave room in LDS for
//   one workgroup: as many waves share them as their queues leave room for.
// (4, 4) and (1, 16): few workgroups.  A scan of m candidates is a chain of m
//   steps however many compute units are idle; splitting it over S waves and
//   merging their lists (list_merge, log2 S rounds through LDS) shortens it.
//   (1, 16) writes tables only: a sweep's co-moments are merged per 256 queries.
// Merge of the S lists of every query into the lists of split 0: in each
// round the upper half of the splits left writes its lists to LDS.
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
constexpr int64_t kScanLdsMax = 160 * 1024 - 4608;  // less the kernels' static LDS
template <int Q, int S>
constexpr int64_t scan_lds(int64_t /*L_max*/, int K, int64_t lds_x) {
  const int64_t queue = static_cast<int64_t>(Q) * S * kPendBytes;
  const int64_t merge = merge_bytes<Q, S>(K);
  return lds_x * 4 + (queue > merge ? queue : merge);
}

enum class ScanLayout { kPlain, kLong8, kLong16, kSplit4, kTable16 };
constexpr int kCus = 256;  // compute units of the chip
constexpr int64_t kTable16Groups = kCus;
constexpr int64_t kSplit4Blocks = 2 * kCus;
constexpr int64_t kLongSeries = 8192;  // above, 160 KB of LDS hold fewer than three workgroups of four waves

// Layout of a launch over nslots series of up to L_max samples and lists of K
// entries (wants_mom: the launch writes a sweep's co-moments).
inline ScanLayout scan_layout(int64_t nslots, int64_t L_max, int K, bool wants_mom) {
  const int64_t lds_x = L_max + 138;  // (scan_floats)
  const int64_t groups = (L_max + 63) / 64 * nslots, blocks = (L_max + 255) / 256 * nslots;
  if (!wants_mom && groups <= kTable16Groups && scan_lds<1, 16>(L_max, K, lds_x) <= kScanLdsMax)
    return ScanLayout::kTable16;
  if (blocks <= kSplit4Blocks && scan_lds<4, 4>(L_max, K, lds_x) <= kScanLdsMax) return ScanLayout::kSplit4;
  if (L_max > kLongSeries && scan_lds<16, 1>(L_max, K, lds_x) <= kScanLdsMax) return ScanLayout::kLong16;
  if (L_max > kLongSeries && scan_lds<8, 1>(L_max, K, lds_x) <= kScanLdsMax) return ScanLayout::kLong8;
  return ScanLayout::kPlain;
}

}  // namespace edm
