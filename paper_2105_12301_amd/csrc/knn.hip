// All-kNN scans with lag 1 or E = 1 (knn_kernel.h) and the dispatch over lags.
#include <array>
#include <utility>

#include "knn_kernel.h"

namespace edm {
namespace {

using LaunchFn = hipError_t (*)(const KnnArgs &, int, int64_t, hipStream_t);

template <size_t... I>
constexpr auto make_fast(std::index_sequence<I...>) {
  return std::array<LaunchFn, sizeof...(I)>{
      &launch_layout<static_cast<int>(I) + 1, static_cast<int>(I) + 2, true>...};
}

}  // namespace

// (The filter takes longer at every E: 16384 samples E = 5, 12, 20 142, 251, 423 us
// split, 429, 518, 706 through the filter; 300 samples 14, 20, 28 against 30, 93, 79.)
bool knn_splits(int64_t L) { return scan_layout(1, L, EDM_E_MAX, EDM_E_MAX + 1, false) == ScanLayout::kTableSplit; }

hipError_t launch_knn_scan(const KnnArgs &a, int nslots, int64_t L_max, hipStream_t st) {
  static const auto fast = make_fast(std::make_index_sequence<EDM_E_MAX>{});
  if (nslots <= 0) return hipSuccess;
  KnnArgs b = a;
  b.lds_x = scan_floats(L_max);
  // (E = 1 has no lag, and every lag is allowed with it: never a lagged scan)
  if ((a.tau == 1 || a.E == 1) && a.k == a.E + 1 && a.E >= 1 && a.E <= EDM_E_MAX) return fast[a.E - 1](b, nslots, L_max, st);
  return launch_knn_lagged(b, nslots, L_max, st);
}

hipError_t launch_knn(const KnnArgs &a, int nslots, int64_t L_max, hipStream_t st) {
  if (nslots <= 0) return hipSuccess;
  TimedLaunch timed(EDM_KF_EXACT_SCAN, st);
  return launch_knn_scan(a, nslots, L_max, st);
}

}  // namespace edm
