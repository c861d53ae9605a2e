// Cross-map tables from the E sweep's neighbour lists (kEDM paper: Section
// 3.4 runs the simplex E sweep and then the cross map of every pair at the
// target's E; both need every library's k-nearest-neighbour table at that E).
//
// The sweep predicts Tp = 1 ahead: at dimension E (tau = 1) its queries and
// candidates are the m1 = L - E first embedded points.  The cross map at
// Tp = 0 has m0 = m1 + 1 of each: one more candidate, index m1, and one more
// query, p = m1.  For p < m1 the Tp = 0 list is therefore the sweep's list
// with candidate m1 offered last; it has the largest index, so a strict "<"
// puts it after equal keys, exactly where a full scan would (and where it
// does not enter, the sweep's weights are the table's).  Query p = m1 is
// scanned in full.  A series with no sweep list at E (m1 - 1 < E + 1) but
// a defined cross map (m0 - 1 >= E + 1) has every query scanned.
// Keys are the float32 sums of Algorithm 1 (contraction off), so the tables
// are bit-identical to the scans'.
#include <array>
#include <utility>

#include "../../include/edm.h"
#include "device_common.h"
#include "kernels.h"
#include "scan_common.h"

#pragma clang fp contract(off)

namespace edm {
namespace {

template <int E>
__device__ __forceinline__ float canon_key(const float *__restrict__ xs, int p, int q) {
  float acc = 0.0f;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const float d = xs[p + j] - xs[q + j];
    acc = acc + d * d;
  }
  return acc;
}

__device__ __forceinline__ void stage(const KnnArgs &a, int row, int L, float *xs) {
  const float *__restrict__ x = a.X + static_cast<int64_t>(row) * a.ldx;
  for (int i = threadIdx.x; i < L; i += blockDim.x) xs[i] = x[i];
  __syncthreads();
}

// Queries p < m1: one thread per query, the series read from global memory
// (L2).  The sweep's list is the cross map's unless candidate m1 enters it,
// that is unless key(p, m1) < key(p, last entry); then the list and the
// weights the sweep kept are the table row (the weights depend only on the
// query and its neighbours), and when the table is the kept array itself the
// row is left as it is.  Otherwise (about one query in a hundred) the query
// is queued in LDS, and the queue is worked off by consecutive threads: every
// key is recomputed, m1 is inserted and the row is rewritten (the kept
// entries are read before).
template <int E>
__device__ __forceinline__ void fix_block(const KnnArgs &a, int row, int (&queue)[256], int &n_queue) {
  constexpr int K = E + 1;
  if (a.group_at && a.group_at[E + 1] == a.group_at[E]) return;  // no target of this E
  const int L = static_cast<int>(a.L_dev ? a.L_dev[row] : a.L_uni);
  const int m1 = L - E;
  if (m1 - 1 < K) return;  // no sweep list: k_scan_queries covers this series
  if (static_cast<int>(blockIdx.x) * 256 >= m1) return;  // (uniform)
  const float *__restrict__ x = a.X + static_cast<int64_t>(row) * a.ldx;
  auto key_of = [&](int p, int q) {
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const float d = x[p + j] - x[q + j];
      acc = acc + d * d;
    }
    return acc;
  };
  // Queries where m1 enters the list (about 1 in 100) are queued in LDS and
  // rewritten by consecutive threads, so the slow path runs on few waves.
  if (threadIdx.x == 0) n_queue = 0;
  __syncthreads();
  const int p = static_cast<int>(blockIdx.x) * 256 + static_cast<int>(threadIdx.x);
  const bool same = a.idxE[E] == a.keepE[E] && a.wE[E] == a.keepWE[E] && a.strideE[E] == a.keep_strideE[E];
  if (p < m1) {
    const int64_t ko = static_cast<int64_t>(row) * a.keep_strideE[E] + static_cast<int64_t>(p) * K;
    const int32_t *__restrict__ kp = a.keepE[E] + ko;
    if (a.keepWE[E] && !(key_of(p, m1) < key_of(p, kp[K - 1]))) {
      // the kept row is the table row: nothing to do when the table is the
      // kept array itself (one extra row per slot for query m1), else a copy
      if (!same) {
        const int64_t base = static_cast<int64_t>(row) * a.strideE[E] + static_cast<int64_t>(p) * K;
        const float *__restrict__ kw = a.keepWE[E] + ko;
#pragma unroll
        for (int i = 0; i < K; ++i) {
          a.idxE[E][base + i] = kp[i];
          a.wE[E][base + i] = kw[i];
        }
      }
    } else {
      queue[atomicAdd(&n_queue, 1)] = p;
    }
  }
  __syncthreads();
  const int nq = n_queue;
  for (int i = static_cast<int>(threadIdx.x); i < nq; i += 256) {
    const int pq = queue[i];
    const int32_t *__restrict__ kp =
        a.keepE[E] + static_cast<int64_t>(row) * a.keep_strideE[E] + static_cast<int64_t>(pq) * K;
    float vp[E];
#pragma unroll
    for (int j = 0; j < E; ++j) vp[j] = x[pq + j];
    const float k_m1 = key_of(pq, m1);
    // m1 enters after every entry whose key is at most its own (it has the
    // largest index) and pushes the last entry out.
    int pos = 0;
#pragma unroll 1
    for (int r = 0; r < K; ++r) pos += key_of(pq, kp[r]) <= k_m1 ? 1 : 0;
    int qi[K];
#pragma unroll
    for (int r = 0; r < K; ++r) qi[r] = r < pos ? kp[r] : (r == pos ? m1 : kp[r - 1 < 0 ? 0 : r - 1]);
    finish_list<E, E>(a, row, pq, L, 0, 1u << (E - 1), vp, qi, x);
  }
}

template <int E>
__global__ __launch_bounds__(256) void k_fix_from_sweep(KnnArgs a, int slot0) {
  __shared__ int queue[256];
  __shared__ int n_queue;
  fix_block<E>(a, slot0 + static_cast<int>(blockIdx.y), queue, n_queue);
}

// Full scans, one query per wave: the lanes walk the candidates in ascending
// order keeping their own sorted lists, then the K smallest (key, index) of
// the 64 lists are taken one at a time (lexicographic, ties to the lower
// index).  Query m1 of every series, or every query of a series whose sweep
// had no list at E.
template <int E>
__device__ __forceinline__ void scan_block(const KnnArgs &a, int row, float *fx_xs) {
  constexpr int K = E + 1;
  if (a.group_at && a.group_at[E + 1] == a.group_at[E]) return;  // no target of this E
  const int L = static_cast<int>(a.L_dev ? a.L_dev[row] : a.L_uni);
  const int m0 = L - (E - 1), m1 = m0 - 1;
  if (m0 - 1 < K) return;  // the cross map is undefined at E for this library
  stage(a, row, L, fx_xs);
  const int wave = static_cast<int>(threadIdx.x) / kWave;
  const int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
  const int p_first = (m1 - 1 < K) ? 0 : m1;
  for (int p = p_first + wave; p < m0; p += static_cast<int>(blockDim.x) / kWave) {
    double l[K];
#pragma unroll
    for (int i = 0; i < K; ++i) l[i] = entry_empty();
    for (int q = lane; q < m0; q += kWave) {
      const float kq = q == p ? __builtin_inff() : canon_key<E>(fx_xs, p, q);
      if (kq < entry_key(l[K - 1])) list_insert<0, K, K>(l, entry(kq, q));
    }
    int ri[K];
#pragma unroll
    for (int r = 0; r < K; ++r) {
      double best = l[0];
#pragma unroll
      for (int m = 1; m < kWave; m <<= 1) best = entry_min(best, __shfl_xor(best, m));
      ri[r] = entry_idx(best);
      if (entry_idx(l[0]) == ri[r]) {  // this lane held the winner (or is empty): drop it
#pragma unroll
        for (int i = 0; i < K - 1; ++i) l[i] = l[i + 1];
        l[K - 1] = entry_empty();
      }
    }
    if (lane == 0) {
      float vp[E];
#pragma unroll
      for (int j = 0; j < E; ++j) vp[j] = fx_xs[p + j];
      finish_list<E, E>(a, row, p, L, 0, 1u << (E - 1), vp, ri, fx_xs);
    }
  }
}

template <int E>
__global__ __launch_bounds__(256) void k_scan_queries(KnnArgs a, int slot0) {
  extern __shared__ float fx_xs[];
  scan_block<E>(a, slot0 + static_cast<int>(blockIdx.y), fx_xs);
}

// Both for every E at once (blockIdx.z): few series, where each of the 2 E_max
// launches would take a few microseconds and find most buckets empty.  The two
// write different rows and read only the series and the sweep's lists.
template <int... I>
__device__ __forceinline__ void tables_block(const KnnArgs &a, int E, float *xs, int (&queue)[256], int &n_queue,
                                             std::integer_sequence<int, I...>) {
  const int row = static_cast<int>(blockIdx.y);
  if (blockIdx.x + 1 < gridDim.x)
    ((E == I + 1 ? fix_block<I + 1>(a, row, queue, n_queue) : void()), ...);
  else
    ((E == I + 1 ? scan_block<I + 1>(a, row, xs) : void()), ...);
}
__global__ __launch_bounds__(256) void k_tables_all(KnnArgs a) {
  extern __shared__ float fx_xs[];
  __shared__ int queue[256];
  __shared__ int n_queue;
  tables_block(a, static_cast<int>(blockIdx.z) + 1, fx_xs, queue, n_queue,
               std::make_integer_sequence<int, EDM_E_MAX>{});
}

using FixFn = hipError_t (*)(const KnnArgs &, int, int64_t, hipStream_t);

template <int E>
hipError_t launch_fix(const KnnArgs &a, int nslots, int64_t L_max, hipStream_t st) {
  const size_t shm = static_cast<size_t>(L_max) * sizeof(float);
  const void *f2 = reinterpret_cast<const void *>(&k_scan_queries<E>);
  if (shm > 65536) {
    hipError_t e = hipFuncSetAttribute(f2, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(shm));
    if (e != hipSuccess) return e;
  }
  const unsigned gx = static_cast<unsigned>((L_max + 255) / 256);
  constexpr int kMaxY = 32768;
  for (int s0 = 0; s0 < nslots; s0 += kMaxY) {
    const unsigned ny = static_cast<unsigned>(nslots - s0 < kMaxY ? nslots - s0 : kMaxY);
    hipLaunchKernelGGL(k_fix_from_sweep<E>, dim3(gx, ny), dim3(256), 0, st, a, s0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_queries<E>, dim3(1, ny), dim3(256), shm, st, a, s0);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <size_t... I>
constexpr std::array<FixFn, EDM_E_MAX> fix_table(std::index_sequence<I...>) {
  return {{&launch_fix<static_cast<int>(I) + 1>...}};
}

}  // namespace

hipError_t launch_tables_from_sweep_all(const KnnArgs &a, int E_max, int nslots, int64_t L_max, hipStream_t st) {
  if (E_max < 1 || E_max > EDM_E_MAX || nslots > 65535 || a.tau != 1 || a.mom != nullptr) return hipErrorInvalidValue;
  if (nslots <= 0) return hipSuccess;
  const size_t shm = static_cast<size_t>(L_max) * sizeof(float);
  if (shm > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_tables_all),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(shm));
    if (e != hipSuccess) return e;
  }
  TimedLaunch timed(EDM_KF_TABLES_FROM_SWEEP, st);
  const dim3 grid(static_cast<unsigned>((L_max + 255) / 256 + 1), static_cast<unsigned>(nslots),
                  static_cast<unsigned>(E_max));
  hipLaunchKernelGGL(k_tables_all, grid, dim3(256), shm, st, a);
  return hipGetLastError();
}

hipError_t launch_tables_from_sweep(const KnnArgs &a, int E, int nslots, int64_t L_max,
                                    hipStream_t st) {
  static const std::array<FixFn, EDM_E_MAX> t = fix_table(std::make_index_sequence<EDM_E_MAX>{});
  if (E < 1 || E > EDM_E_MAX || a.tau != 1 || a.mom != nullptr || !a.keepE[E] || !a.idxE[E] ||
      !a.wE[E])
    return hipErrorInvalidValue;
  if (nslots <= 0) return hipSuccess;
  TimedLaunch timed(EDM_KF_TABLES_FROM_SWEEP, st);
  return t[E - 1](a, nslots, L_max, st);
}

}  // namespace edm
