// Register top-k lists and the per-E epilogue shared by the batched scans
// (exact VALU scan in sweep_multi.hip, matrix-core filter in gram.hip).
// Every file that includes this header is compiled with FP contraction off.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "../../include/edm.h"
#include "device_common.h"
#include "kernels.h"
#include "topk_list.h"

namespace edm {

template <int I0, int I1, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I0 <= I1) {
    f(std::integral_constant<int, I0>{});
    static_for<I0 + 1, I1>(f);
  }
}

// Offset of dimension E's list inside the flat register arrays of a group
// whose smallest dimension is ELO (list of E holds E + 1 entries).
template <int ELO>
constexpr int list_off(int E) {
  int o = 0;
  for (int e = ELO; e < E; ++e) o += e + 1;
  return o;
}

// Staged series of an exact scan: zeros before and after the samples, so the
// first and last steps of the diagonal order need no clamped addresses.
constexpr int kScanFront = 64;  // lane l sees candidate s + l from s = -63 on
constexpr int kScanBack = 72;   // ... up to s + l = L + 62, plus one unrolled block
constexpr int kScanUnroll = 8;  // steps per block

// Floats of LDS for a staged series of up to L_max samples (even: 8-byte queue
// entries follow).
inline int32_t scan_floats(int64_t L_max) {
  return static_cast<int32_t>((L_max + kScanFront + kScanBack + 1) / 2 * 2);
}

// Stages x[0, L) at smem + kScanFront with its pads; ends with a barrier.
template <int kT>
__device__ __forceinline__ float *stage_scan(const float *__restrict__ x, int L, float *smem, int *status) {
  float *xs = smem + kScanFront;
  bool bad = false;
  for (int i = static_cast<int>(threadIdx.x) - kScanFront; i < L + kScanBack; i += kT) {
    float v = 0.0f;
    if (i >= 0 && i < L) {
      v = x[i];
      bad |= !isfinite(v);
    }
    xs[i] = v;
  }
  if (bad) atomicOr(status, 1);
  __syncthreads();
  return xs;
}

// The candidate steps of one wave in diagonal order: at step s lane l sees
// candidate q = s + l.  Steps [s0, s_end) of the range -63 .. m - 1; the steps
// of one residue modulo tau share samples, so a window of EHI + 7 of them
// slides along in registers, one LDS word per candidate.  Calls
// visit(s, q, key, edge): key[E - ELO] for every E of [ELO, EHI] (Algorithm 1,
// one running float32 sum); edge: a constant type that says whether q (or
// step s) may lie outside the range.  check() after every kCheck steps.
// s_full: steps at or beyond it may be out of range.
template <int ELO, int EHI, bool T1, int kCheck, class Visit, class Check>
__device__ __forceinline__ void scan_steps(const float (&vp)[EHI], const float *xs, int lane, int tau_, int s0,
                                           int s_end, int s_full, Visit &&visit, Check &&check) {
  constexpr int U = kScanUnroll;
  constexpr int NG = EHI - ELO + 1;
  const int tau = T1 ? 1 : tau_;
  auto block = [&](int s, const float (&win)[EHI + U - 1], auto edge) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float acc = 0.0f;
      float key[NG];
      static_for<0, EHI - 1>([&](auto JC) {
        constexpr int j = decltype(JC)::value;
        const float d = vp[j] - win[u + j];
        acc = acc + d * d;
        if constexpr (j + 1 >= ELO) key[j + 1 - ELO] = acc;
      });
      visit(s + u * tau, s + u * tau + lane, key, edge);
      if ((u + 1) % kCheck == 0) check();
    }
  };
#pragma unroll 1
  for (int r = 0; r < tau && s0 + r < s_end; ++r) {
    int s = s0 + r;
    // with tau = 1 the last block may pass s_end (its steps are masked)
    const int s_last = T1 ? s_end : s_end - (U - 1) * tau;
    if (s < s_last) {
      float win[EHI + U - 1];
#pragma unroll
      for (int j = 0; j < EHI - 1; ++j) win[j] = xs[s + lane + j * tau];
      auto run = [&](int lim, auto edge) {
#pragma unroll 1
        for (; s < lim; s += U * tau) {
#pragma unroll
          for (int u = 0; u < U; ++u) win[EHI - 1 + u] = xs[s + lane + (EHI - 1 + u) * tau];
          block(s, win, edge);
#pragma unroll
          for (int j = 0; j < EHI - 1; ++j) win[j] = win[j + U];
        }
      };
      run(s_last < 0 ? s_last : 0, std::true_type{});
      run(s_full - (U - 1) * tau, std::false_type{});
      run(s_last, std::true_type{});
    }
    if constexpr (!T1) {
#pragma unroll 1
      for (; s < s_end; s += tau) {  // remainder of the residue
        float acc = 0.0f;
        float key[NG];
        static_for<0, EHI - 1>([&](auto JC) {
          constexpr int j = decltype(JC)::value;
          const float d = vp[j] - xs[s + lane + j * tau];
          acc = acc + d * d;
          if constexpr (j + 1 >= ELO) key[j + 1 - ELO] = acc;
        });
        visit(s, s + lane, key, std::true_type{});
        check();
      }
    }
  }
}

// Final step for dimension E of query p: float64 distances and weights of the
// K = E + 1 winners (Section 2.1 step 3, "Normalize D_k" of Algorithm 2),
// then either the table row (table mode) or the query's self-prediction Tp
// ahead (sweep mode, returned as a one-point moment).  vp holds the query's
// samples, xs the staged series, qi the neighbours in list order (consumed).
template <int E, int NV>
__device__ __forceinline__ Mom finish_list(const KnnArgs &a, int row, int p, int L, int Tp,
                                           uint32_t need, const float (&vp)[NV],
                                           int (&qi)[E + 1], const float *__restrict__ xs) {
  constexpr int K = E + 1;
  const int mE = L - (E - 1) - Tp;
  Mom mine = mom_zero();
  const bool want_table = a.mom == nullptr && ((need >> (E - 1)) & 1u);
  if (p < mE && mE - 1 >= K && (a.mom != nullptr || want_table)) {
    double D[K];
    double dmin = __builtin_inf();
#pragma unroll 1
    for (int r = 0; r < K; ++r) {
      const int q = qi[0] < 0 ? 0 : qi[0];
      double s2 = 0.0;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const double d = static_cast<double>(vp[j]) - static_cast<double>(xs[q + j]);
        s2 += d * d;
      }
      const double dq = sqrt(s2);
      dmin = fmin(dmin, dq);
#pragma unroll
      for (int i = 0; i < K - 1; ++i) {
        qi[i] = qi[i + 1];
        D[i] = D[i + 1];
      }
      qi[K - 1] = q;
      D[K - 1] = dq;
    }
    double wsum = 0.0;
#pragma unroll 1
    for (int r = 0; r < K; ++r) {
      const double d = D[0];
      const double wq = dmin > 0.0 ? exp(-d / dmin) : (d == 0.0 ? 1.0 : 0.0);
      wsum += wq;
#pragma unroll
      for (int i = 0; i < K - 1; ++i) D[i] = D[i + 1];
      D[K - 1] = wq;
    }
    const double inv = 1.0 / wsum;
    if (want_table) {
      int32_t *ti;
      float *tw;
      int64_t base;
      if (a.tbl_off) {
        const int64_t o = a.tbl_off[static_cast<int64_t>(row) * (EDM_E_MAX + 1) + E];
        ti = a.tbl_idx + o;
        tw = a.tbl_w + o;
        base = static_cast<int64_t>(p) * K;
      } else {
        ti = a.idxE[E];
        tw = a.wE[E];
        base = static_cast<int64_t>(row) * a.strideE[E] + static_cast<int64_t>(p) * K;
      }
#pragma unroll
      for (int i = 0; i < K; ++i) {
        ti[base + i] = qi[i];
        tw[base + i] = static_cast<float>(D[i] * inv);
      }
    } else {
      if (a.keepE[E]) {  // sweep mode: keep the sorted list for a later cross map
        const int64_t ko = static_cast<int64_t>(row) * a.keep_strideE[E] + static_cast<int64_t>(p) * K;
#pragma unroll
        for (int i = 0; i < K; ++i) a.keepE[E][ko + i] = qi[i];
        if (a.keepWE[E]) {
#pragma unroll
          for (int i = 0; i < K; ++i) a.keepWE[E][ko + i] = static_cast<float>(D[i] * inv);
        }
      }
      const int o_off = (E - 1) + Tp;
      double yh = 0.0;
#pragma unroll
      for (int i = 0; i < K; ++i) yh += (D[i] * inv) * static_cast<double>(xs[qi[i] + o_off]);
      mine.n = 1.0;
      mine.mo = static_cast<double>(xs[p + o_off]);
      mine.mp = yh;
    }
  }
  return mine;
}

}  // namespace edm
