// All-kNN scans with a lag above 1, and with any number of neighbours
// (knn_kernel.h): a translation unit of their own for the build's sake.
#include <array>
#include <utility>

#include "knn_kernel.h"

namespace edm {
namespace {

using LaunchFn = hipError_t (*)(const KnnArgs &, int, int64_t, hipStream_t);

template <int K>
hipError_t launch_generic(const KnnArgs &a, int nslots, int64_t L_max, hipStream_t st) {
  if (a.mom == nullptr && (L_max + 63) / 64 * nslots <= kTableSplitGroups &&
      scan_lds<1, 16>(K, a.lds_x, true) <= kScanLdsMax)
    return launch_one<0, K, false, 1, 16, true>(a, nslots, L_max, st);
  return launch_one<0, K, false, 4, 1, false>(a, nslots, L_max, st);
}

template <size_t... I>
constexpr auto make_lagged(std::index_sequence<I...>) {
  return std::array<LaunchFn, sizeof...(I)>{
      &launch_layout<static_cast<int>(I) + 2, static_cast<int>(I) + 3, false>...};  // from E = 2
}
template <size_t... I>
constexpr auto make_generic(std::index_sequence<I...>) {
  return std::array<LaunchFn, sizeof...(I)>{&launch_generic<static_cast<int>(I) + 1>...};
}

}  // namespace

hipError_t launch_knn_lagged(const KnnArgs &a, int nslots, int64_t L_max, hipStream_t st) {
  static const auto lagged = make_lagged(std::make_index_sequence<EDM_E_MAX - 1>{});
  static const auto generic = make_generic(std::make_index_sequence<EDM_K_MAX>{});
  const bool fast = a.k == a.E + 1 && a.E >= 2 && a.E <= EDM_E_MAX;
  return fast ? lagged[a.E - 2](a, nslots, L_max, st) : generic[a.k - 1](a, nslots, L_max, st);
}

}  // namespace edm
