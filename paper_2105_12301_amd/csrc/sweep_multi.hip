// Batched E sweep: one candidate scan serves a whole group of embedding
// dimensions (kEDM paper: Section 2.1 steps 1-4 with E chosen empirically,
// Algorithms 1-2; the batching over E is this library's own).
//
// The ranking key of Algorithm 1 for dimension E is the float32 sum over the
// lags j < E in ascending order, so the key for E is exactly the key for E-1
// plus one more rounded term.  A lane that owns query p therefore walks its
// candidates once, extends the running sum lag by lag, and offers the partial
// sum to the top-k list of every E in its group as it passes: the tables (and
// so the correlations) are bit-identical to one scan per E, for
// 3*E_hi + (E_hi - E_lo + 1) VALU ops per pair instead of sum_E (3E + 1).
//
// Everything else follows the per-E kernel in knn_kernel.h: library staged in
// LDS, one query per lane, diagonal candidate order (lane l sees q = s + l), a
// sliding window of samples in registers, improving candidates queued in LDS
// and inserted in batches where that pays (10000 x 2000, Tp = 1: E 1-4 27.2 -> 21
// ms, all five groups 453 -> 388 ms against insertion as they come), float64 weights of
// the winners, the self-prediction and its Pearson
// co-moments reduced per block.  tau = 1 only (the sweep's lag); other lags
// use the per-E kernel.
#include <array>
#include <utility>

#include "../../include/edm.h"
#include "device_common.h"
#include "kernels.h"
#include "group_scan.h"
#include "scan_common.h"

#pragma clang fp contract(off)

namespace edm {
namespace {

template <int ELO, int EHI, int Q, int S, bool kQueue>
__global__ __launch_bounds__(kWave * Q * S) void k_sweep_multi(KnnArgs a, int slot0) {
  extern __shared__ __attribute__((aligned(16))) float scan_smem[];
  group_scan<ELO, EHI, Q, S, kQueue>(a, slot0 + static_cast<int>(blockIdx.y), static_cast<int>(blockIdx.x), scan_smem);
}

// Persistent form: each workgroup pulls (row, block) items of one E group,
// ordered by the host longest first, from a device counter until the list is
// exhausted (every workgroup reaches the exit).  The item index travels
// through LDS and is made wave-uniform.
template <int ELO, int EHI, int Q, bool kQueue, bool kGate>
__global__ __launch_bounds__(kWave * Q) void k_tables_persistent(KnnArgs a, const TableItem *__restrict__ items,
                                                                 int n_items, int *counter) {
  extern __shared__ __attribute__((aligned(16))) float scan_smem[];
  __shared__ int item_s;
  for (int trip = 0;; ++trip) {  // one call site for the body (see lookup.hip)
    int it;
    if (counter == nullptr) {  // one item per workgroup
      if (trip > 0) break;
      it = static_cast<int>(blockIdx.x);
    } else {
      __syncthreads();  // the previous item is done with xs and item_s
      if (threadIdx.x == 0) item_s = atomicAdd(counter, 1);
      __syncthreads();
      it = __builtin_amdgcn_readfirstlane(item_s);
      if (it >= n_items) break;
    }
    const int row = __builtin_amdgcn_readfirstlane(items[it].row);
    const int blk = __builtin_amdgcn_readfirstlane(static_cast<int>(items[it].blk));
    group_scan<ELO, EHI, Q, 1, kQueue, kGate>(a, row, blk / (Q / 4), scan_smem);  // (blk: a multiple of Q / 4)
  }
}

// Groups of E sharing one scan: the register lists of a group hold at most
// ~54 entries (108 VGPRs).
constexpr int kGroups[][2] = {{1, 8}, {9, 12}, {13, 15}, {16, 18}, {19, 20}};

// Workgroup of a group scan without splits: Q waves, queued or not.
// Groups of several E beyond 4 are queued (inserting as candidates come runs
// nearly every list on nearly every step: E 1-8 of 1000 x 1000 1593 us queued,
// 3683 not), by as many waves as leave the most in flight (most_resident: E 1-8
// of 300 x 12000 39.7 ms by 4 waves, 41.6 by 8; 100 x 20000 67.6 and 36.0).
// A group of one E follows queue_wins.  E 1-2 never queue (2000 x 2000 2.24 ms
// against 2.47 queued), E 1-3 and 1-4 up to 3000 and 6000 samples (queued / not:
// E 1-3 3.17 / 3.51 at 2000, 4.51 / 4.12 at 5000; E 1-4 5.45 / 5.60 at 512 x 5000,
// 7.61 / 6.53 at 256 x 8000).
struct GroupShape {
  int Q;
  bool queue;
};
template <int ELO, int EHI>
constexpr bool group_queues(int64_t L_max) {
  if (ELO == EHI) return queue_wins(ELO, L_max);
  return EHI > 4 || (EHI == 4 && L_max <= 6000) || (EHI == 3 && L_max <= 3000);
}
// Waves a CU holds by the registers of the group's kernel (E 1-2, 1-3: 32, but 16
// waves a workgroup for them were slower: 9.98 against 9.52 ms at 100 x 20000).
template <int ELO, int EHI>
constexpr int group_wave_cap() {
  constexpr int entries = list_off<ELO>(EHI + 1);
  if (ELO == EHI) return scan_wave_cap(ELO);
  if (EHI <= 4) return 24;
  if (entries <= 21 || EHI <= 7) return 16;
  return EHI <= 12 || (EHI <= 17 && entries <= 35) ? 12 : 8;
}
// All LDS of a workgroup: the series, the queues, the waves' co-moments.
template <int ELO, int EHI, bool kQueue>
constexpr int64_t group_lds(int Q, int64_t L_max) {
  const size_t queue = Q * group_extra_lds<ELO, EHI, 4, 1, kQueue>() / 4;
  return (L_max + 138) * 4 + static_cast<int64_t>(queue) + 48 * Q * (EHI - ELO + 1) + 16;
}
template <int ELO, int EHI>
GroupShape group_shape(int64_t L_max, int64_t blocks) {
  constexpr int cap = group_wave_cap<ELO, EHI>();
  const bool few = EHI <= 4 || ELO == EHI;  // may run without queues
  if (few && group_queues<ELO, EHI>(L_max)) return {4, true};
  if (few)
    return {most_resident(EHI <= 4 ? 16 : 8, cap, blocks, [&](int q) { return group_lds<ELO, EHI, false>(q, L_max); }),
            false};
  return {most_resident(8, cap, blocks, [&](int q) { return group_lds<ELO, EHI, true>(q, L_max); }), true};
}
// Calls f(Q, queue) with the shape as constants, for the shapes group_shape gives.
template <int ELO, int EHI, class F>
auto with_shape(GroupShape s, F &&f) {
  using std::bool_constant;
  using std::integral_constant;
  constexpr bool few = EHI <= 4 || ELO == EHI, queued = !few || (ELO == EHI ? ELO >= kQueueE : EHI >= 3);
  if constexpr (queued) {
    if (s.queue && (few || s.Q == 4)) return f(integral_constant<int, 4>{}, bool_constant<true>{});
  }
  if constexpr (!few) return f(integral_constant<int, 8>{}, bool_constant<true>{});
  if constexpr (few) {
    if constexpr (EHI <= 4) {
      if (s.Q == 16) return f(integral_constant<int, 16>{}, bool_constant<false>{});
    }
    if (s.Q == 8) return f(integral_constant<int, 8>{}, bool_constant<false>{});
    return f(integral_constant<int, 4>{}, bool_constant<false>{});
  }
}

template <class F>
hipError_t allow_lds(F fn, size_t shm) {
  if (shm <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                             static_cast<int>(shm));
}

template <int ELO, int EHI, int Q, int S, bool kQueue>
hipError_t launch_group_q(const KnnArgs &a, int nslots, int64_t L_max, hipStream_t st) {
  const size_t shm = static_cast<size_t>(a.lds_x) * sizeof(float) + group_extra_lds<ELO, EHI, Q, S, kQueue>();
  hipError_t e = allow_lds(&k_sweep_multi<ELO, EHI, Q, S, kQueue>, shm);
  if (e != hipSuccess) return e;
  const unsigned gx = static_cast<unsigned>((L_max + kWave * Q - 1) / (kWave * Q));
  constexpr int kMaxY = 32768;
  for (int s0 = 0; s0 < nslots; s0 += kMaxY) {
    const int ny = nslots - s0 < kMaxY ? nslots - s0 : kMaxY;
    hipLaunchKernelGGL((k_sweep_multi<ELO, EHI, Q, S, kQueue>), dim3(gx, static_cast<unsigned>(ny)),
                       dim3(kWave * Q * S), shm, st, a, s0);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

using LaunchFn = hipError_t (*)(const KnnArgs &, int, int64_t, hipStream_t);

template <int ELO, int EHI>
hipError_t launch_group(const KnnArgs &a, int nslots, int64_t L_max, hipStream_t st) {
  const int64_t blocks = (L_max + 255) / 256 * nslots;
  if constexpr (EHI <= 4) {  // (larger groups' lists do not fit the registers of 16 waves)
    constexpr bool kQueue = EHI > 1;
    if (blocks <= split_blocks(EHI, L_max) &&
        a.lds_x * 4 + static_cast<int64_t>(group_extra_lds<ELO, EHI, 4, 4, kQueue>()) <= kScanLdsMax)
      return launch_group_q<ELO, EHI, 4, 4, kQueue>(a, nslots, L_max, st);
  }
  return with_shape<ELO, EHI>(group_shape<ELO, EHI>(L_max, blocks), [&](auto QC, auto queue) {
    return launch_group_q<ELO, EHI, decltype(QC)::value, 1, decltype(queue)::value>(a, nslots, L_max, st);
  });
}

// table[lo-1][hi-lo]: every (lo, hi) with lo a group start and hi inside it.
template <int LO, size_t... I>
constexpr std::array<LaunchFn, 8> row_for(std::index_sequence<I...>) {
  return {{&launch_group<LO, LO + static_cast<int>(I)>...}};
}

}  // namespace

hipError_t launch_sweep_multi(const KnnArgs &a, int nslots, int64_t L_max, hipStream_t st) {
  static const std::array<LaunchFn, 8> t1 = row_for<1>(std::make_index_sequence<8>{});
  static const std::array<LaunchFn, 8> t9 = row_for<9>(std::make_index_sequence<4>{});
  static const std::array<LaunchFn, 8> t13 = row_for<13>(std::make_index_sequence<3>{});
  static const std::array<LaunchFn, 8> t16 = row_for<16>(std::make_index_sequence<3>{});
  static const std::array<LaunchFn, 8> t19 = row_for<19>(std::make_index_sequence<2>{});
  if (nslots <= 0) return hipSuccess;
  KnnArgs b = a;
  b.lds_x = scan_floats(L_max);
  // With the matrix-core filter, E >= kGramEMin runs in the filtered groups.
  const bool gram = a.gram_nrm != nullptr && L_max <= kGramLMax;
  // Tables of one E: its own scan.
  auto scan_one = [&](int E) {
    KnnArgs o = b;
    o.E = E;
    o.k = E + 1;
    o.tau = 1;
    o.excl = 0;
    o.idx = a.idxE[E];
    o.w = a.wE[E];
    o.dist = nullptr;
    o.tbl_stride = a.strideE[E];
    TimedLaunch timed(EDM_KF_BATCHED_SCAN, st);
    return launch_knn_scan(o, nslots, L_max, st);
  };
  const bool tables = a.mom == nullptr;
  if (gram && gram_sweep_is_small(nslots, L_max)) {
    // (one E: candidates split over waves take 20-70 us on 8 x 1000, the filter
    // alone 140-230)
    const bool one = tables && a.need != 0 && (a.need & (a.need - 1)) == 0;
    return one ? scan_one(__builtin_ctz(a.need) + 1) : launch_gram_small(a, nslots, L_max, st);
  }
  auto hi_of = [&](int lo, int top) {
    int hi = top < a.E_max ? top : a.E_max;
    if (a.mom == nullptr) {  // table mode: the group's scan must reach its largest needed E
      hi = 0;
      for (int E = lo; E <= top; ++E)
        if ((a.need >> (E - 1)) & 1u) hi = E;
    }
    return hi;
  };
  for (const auto &g : kGroups) {
    const int lo = g[0];
    if (gram && lo >= kGramEMin) break;
    const int top = gram && g[1] >= kGramEMin ? kGramEMin - 1 : g[1];
    const int hi = hi_of(lo, top);
    if (hi == 0) continue;
    if (lo > hi) break;
    const std::array<LaunchFn, 8> &t = lo == 1 ? t1 : lo == 9 ? t9 : lo == 13 ? t13 : lo == 16 ? t16 : t19;
    // Tables of one E, or of two of a larger group, take less one scan each than
    // the group's scan up to the larger one, which inserts into every list (2000 x
    // 2000, group / alone: E 8 8.8 / 4.4 ms, E 15 15.2 / 8.5, E 20 18.3 / 10.9; the
    // whole groups E 9-12, 13-15, 16-18 11.9, 16.8, 20 ms, two of them alone
    // 10-11, 15, 19).  E 1-4 together and E 1 alone do not (E 1-2 2.2 ms, alone 1.6 each).
    uint32_t need = 0;
    for (int E = lo; tables && E <= top; ++E) need |= a.need & (1u << (E - 1));
    const int n = __builtin_popcount(need);
    if ((n == 1 && hi > 1) || (n == 2 && hi > 4 && top - lo > 1)) {
      for (int E = lo; E <= top; ++E) {
        if (!((need >> (E - 1)) & 1u)) continue;
        hipError_t e = scan_one(E);
        if (e != hipSuccess) return e;
      }
      continue;
    }
    TimedLaunch timed(EDM_KF_BATCHED_SCAN, st);
    hipError_t e = t[hi - lo](b, nslots, L_max, st);
    if (e != hipSuccess) return e;
  }
  if (!gram) return hipSuccess;
  for (const auto &g : kGramGroups) {
    const int lo = g[0];
    const int hi = hi_of(lo, g[1]);
    if (hi == 0) continue;
    if (lo > hi) break;
    hipError_t e = launch_gram_group(a, lo, hi, nslots, L_max, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

namespace {

// groups 0-4: the exact E groups; 5: E 1-4 (below the filtered groups)
constexpr int kTables = 6;

using TablesFn = void (*)(KnnArgs, const TableItem *, int, int *);
struct Tables {
  TablesFn fn;
  int waves;
  size_t lds;
};

template <int ELO, int EHI>
Tables tables_of(int64_t L_max, bool gate) {
  constexpr int64_t kMany = int64_t(1) << 40;  // (a work list keeps every CU busy)
  return with_shape<ELO, EHI>(group_shape<ELO, EHI>(L_max, kMany), [&](auto QC, auto queue) {
    constexpr int Q = decltype(QC)::value;
    constexpr bool kQueue = decltype(queue)::value;
    const size_t lds = static_cast<size_t>(scan_floats(L_max)) * sizeof(float) + group_extra_lds<ELO, EHI, Q, 1, kQueue>();
    if constexpr (kQueue && ELO < EHI) {
      if (gate) return Tables{&k_tables_persistent<ELO, EHI, Q, true, true>, Q, lds};
    }
    return Tables{&k_tables_persistent<ELO, EHI, Q, kQueue, false>, Q, lds};
  });
}

Tables tables_for(int group, int64_t L_max, bool gate) {
  switch (group) {
    case 0: return tables_of<1, 8>(L_max, gate);
    case 1: return tables_of<9, 12>(L_max, gate);
    case 2: return tables_of<13, 15>(L_max, gate);
    case 3: return tables_of<16, 18>(L_max, gate);
    case 4: return tables_of<19, 20>(L_max, gate);
    default: return tables_of<1, 4>(L_max, gate);
  }
}

}  // namespace

int tables_item_blocks(int group, int64_t L_max) {
  return group < 0 || group >= kTables ? 1 : tables_for(group, L_max, false).waves / 4;
}

hipError_t launch_tables_persistent(const KnnArgs &a, int group, const TableItem *items,
                                    int n_items, int *counter, int64_t L_max, bool few_needed, int wg_per_cu,
                                    int n_cu, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  if (group < 0 || group >= kTables) return hipErrorInvalidValue;
  KnnArgs b = a;
  b.lds_x = scan_floats(L_max);
  const Tables t = tables_for(group, L_max, few_needed);
  TimedLaunch timed(EDM_KF_BATCHED_SCAN, st);
  hipError_t e = allow_lds(t.fn, t.lds);
  if (e != hipSuccess) return e;
  const dim3 threads(static_cast<unsigned>(kWave * t.waves));
  if (wg_per_cu <= 0) {  // one workgroup per item
    hipLaunchKernelGGL(t.fn, dim3(static_cast<unsigned>(n_items)), threads, t.lds, st, b, items, n_items,
                       static_cast<int *>(nullptr));
    return hipGetLastError();
  }
  int grid = wg_per_cu * n_cu;
  if (grid > n_items) grid = n_items;
  hipLaunchKernelGGL(t.fn, dim3(static_cast<unsigned>(grid)), threads, t.lds, st, b, items, n_items, counter);
  return hipGetLastError();
}

}  // namespace edm
