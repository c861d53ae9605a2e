// All k-nearest-neighbour tables, fused with the time-delay embedding and the
// simplex weights (kEDM paper: Section 2.1 steps 1-3, Algorithms 1 and 2).
//
// Design for gfx950
// -----------------
// * The paper materialises the L x L distance matrix (Algorithm 1) and then
//   partially sorts each row (Algorithm 2).  Here nothing of size L^2 ever
//   leaves the compute unit: each workgroup stages its library series once in
//   LDS (<= 128 KiB of the 160 KiB per CU), each lane owns one query point,
//   keeps its E coordinates and its sorted top-k (key, index) list in VGPRs,
//   and streams every candidate through them.  The embedding is never stored
//   (Section 3.3.1 fuses it for the same reason).
// * Diagonal scan: at step s, lane l of a wave whose queries are p0..p0+63
//   evaluates candidate q = s + l.  Consecutive queries have time-shifted
//   neighbourhoods (v_{p+1} shares E-1 coordinates with v_p), so their top-k
//   insertions fall on the same step and the wave diverges far less often
//   than with every lane looking at the same candidate.  Every lane still
//   visits its candidates in ascending q, so a strict "<" against the k-th key
//   is the whole test (a later equal key has the larger index), and the self
//   step q = p is the same step s = p0 for the whole wave (as is every step of an
//   exclusion window |q - p| <= r: q - p = s - p0 for every lane).
// * tau = 1: each lane keeps a sliding window of E + U - 1 samples in
//   registers and loads one new LDS word per candidate, so the key costs
//   exactly E subtractions, E multiplies and E adds of float32 VALU work.
// * The ranking key is the float32 sum of Algorithm 1 in lag order with a
//   rounding after every operation: this file is compiled with contraction off
//   (and says so with a pragma), and fp32 denormals are kept (gfx950 default).
// * Improving candidates are inserted into the packed lists as they come, or
//   queued in LDS and inserted in batches where that pays (queue_wins in
//   topk_list.h).  What bounds the scan is VALU issue: 3 E + ~20 instructions a
//   step (2000 x 2000, E = 20: 10.9 ms against 6.2 ms for its 61 operations a
//   pair at one a lane and clock; before packed entries 12.5 ms).
// * Few workgroups (one series): the candidates of a query are split over 4 or
//   16 waves whose lists are merged and whose epilogue they share (one series
//   of 1000, E = 3: 86 -> 12 us; 10000 samples, E = 20: 560 us through the filter
//   -> 255 us).
// * Weights need only the k winners: their distances are recomputed in
//   float64 from the staged samples, w_i = exp(-d_i / d_min) normalised
//   (Section 2.1 step 3, "Normalize D_k" in Algorithm 2).
// * Sweep mode fuses the self-prediction and its Pearson co-moments into the
//   epilogue, so the E sweep writes no table at all.
#pragma once

#include "../../include/edm.h"
#include "device_common.h"
#include "kernels.h"
#include "scan_common.h"
#include "topk_list.h"

#pragma clang fp contract(off)

namespace edm {
namespace {

// Waves per SIMD the registers are kept to: four, or three (two) where the list
// and the epilogue's arrays of a scan without splits do not fit 128 (168).
constexpr int knn_waves(int K, int S) { return S > 1 || K <= 17 ? 4 : (K <= 24 ? 3 : 2); }

// Q, S: layout of the workgroup; kQueue: improving candidates are queued (topk_list.h).
template <int E_T, int K, bool T1, int Q, int S, bool kQueue>
__global__ __launch_bounds__(kWave * Q * S, knn_waves(K, S)) void k_knn(KnnArgs a, int slot0) {
  constexpr int EM = E_T ? E_T : EDM_E_MAX;
  constexpr int kT = kWave * Q * S;
  extern __shared__ __attribute__((aligned(16))) float knn_smem[];
  __shared__ Mom wmom[Q];

  const int slot = slot0 + static_cast<int>(blockIdx.y);
  const int row = a.lib_ids ? a.lib_ids[slot] : slot;
  const float *__restrict__ x = a.X + static_cast<int64_t>(row) * a.ldx;
  const int L = static_cast<int>(a.L_dev ? a.L_dev[row] : a.L_uni);
  const int E = E_T ? E_T : a.E;
  const int tau = T1 ? 1 : a.tau;
  const int off = (E - 1) * tau;
  const int m = L - off - a.Tp;  // queries = candidates
  const int excl = a.excl;       // exclusion radius: |q - p| <= excl is no candidate
  if (m - 1 - 2 * excl < K) return;  // infeasible for this series (uniform)
  const int blk0 = static_cast<int>(blockIdx.x) * (kWave * Q);
  if (blk0 >= m) return;

  const float *xs = stage_scan<kT>(x, L, knn_smem, a.status);

  const int lane = threadIdx.x & (kWave - 1);
  // wave-uniform: readfirstlane lets the compiler keep them (and the self step) scalar
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int qg = wave % Q, sp = wave / Q;
  const int p0 = blk0 + qg * kWave;
  const int p = p0 + lane;
  const bool active = p < m;

  float vp[EM];
#pragma unroll
  for (int j = 0; j < EM; ++j) vp[j] = (active && (E_T || j < E)) ? xs[p + j * tau] : 0.0f;

  double l[K];
#pragma unroll
  for (int i = 0; i < K; ++i) l[i] = active ? entry_empty() : entry_idle();
  double *const extra = reinterpret_cast<double *>(knn_smem + a.lds_x);
  Pending pend(extra);
  auto flush = [&]() { pend.drain([&](double e) { list_insert<0, K, K>(l, e); }); };

  if (p0 < m) {  // wave-uniform: a wave with no query skips the scan
    // steps s = -(kWave - 1) .. m - 1; split sp takes one contiguous share
    const int share = (m + kWave - 1 + S - 1) / S;
    const int s0 = -(kWave - 1) + sp * share;
    const int s_end = s0 + share < m ? s0 + share : m;
    auto offer = [&](int s, float acc, int q, bool valid) {
      // T1: a lane's candidates come in ascending q; otherwise the residues
      // are walked one by one and equal keys are ordered by the entry
      if constexpr (kQueue) {
        const bool lt = T1 ? acc < entry_key(l[K - 1]) : entry(acc, q) < l[K - 1];
        pend.push(entry(acc, q), valid && abs(s - p0) > excl && lt);
      } else {
        if (abs(s - p0) <= excl) return;  // (wave-uniform)
        const bool want = valid && (T1 ? acc < entry_key(l[K - 1]) : entry(acc, q) < l[K - 1]);
        if (__builtin_amdgcn_ballot_w64(want)) list_insert<0, K, K>(l, entry(want ? acc : __builtin_inff(), q));
      }
    };
    auto in_range = [&](int s, int q) { return s < s_end && static_cast<unsigned>(q) < static_cast<unsigned>(m); };
    auto check = [&]() {
      if constexpr (kQueue)
        if (pend.full()) flush();
    };
    if constexpr (E_T > 0) {
      const int s_full = m - (kWave - 1) < s_end ? m - (kWave - 1) : s_end;  // below: every lane's q < m
      scan_steps<E_T, E_T, T1, kPendStep>(
          vp, xs, lane, tau, s0, s_end, s_full,
          [&](int s, int q, const float(&key)[1], auto edge) {
            offer(s, key[0], q, !decltype(edge)::value || in_range(s, q));
          },
          check);
    } else {
#pragma unroll 1
      for (int s = s0; s < s_end; ++s) {
        const int q = s + lane;
        const bool valid = in_range(s, q);
        const int qc = valid ? q : 0;
        float acc = 0.0f;
#pragma unroll
        for (int j = 0; j < EM; ++j) {
          if (j >= E) break;  // (uniform: E branches, not 20)
          const float d = vp[j] - xs[qc + j * tau];
          acc = acc + d * d;
        }
        offer(s, acc, q, valid);
        check();
      }
    }
    if constexpr (kQueue) flush();
  }
  // Epilogue: float64 distances of the k winners, weights (Section 2.1 step 3),
  // outputs.  A slot stays unfilled (index 0) only if keys are NaN or overflow to
  // +inf; the status word reports non-finite input.
  Mom mine = mom_zero();
  const int64_t base = static_cast<int64_t>(slot) * a.tbl_stride + static_cast<int64_t>(p) * K;
  auto distance = [&](const float (&v)[EM], int q) {
    double s2 = 0.0;
#pragma unroll
    for (int j = 0; j < EM; ++j) {
      if (E_T || j < E) {
        const double d = static_cast<double>(v[j]) - static_cast<double>(xs[q + j * tau]);
        s2 += d * d;
      }
    }
    return sqrt(s2);
  };
  auto weight = [](double d, double dmin) { return dmin > 0.0 ? exp(-d / dmin) : (d == 0.0 ? 1.0 : 0.0); };
  if constexpr (S > 1) {
    // The S waves of a query share its winners, whose indices, distances and
    // weights pass through LDS (the queues and merges are over): register
    // arrays of them beside the list spill in the 128 registers of a 16-wave
    // workgroup.  Every sum keeps its order.
    merge_splits<Q, S, 0, K, K>(l, extra);
    int32_t *const nbr = reinterpret_cast<int32_t *>(extra + Q * K * kWave) + qg * K * kWave + lane;
    double *const D = extra + qg * K * kWave + lane;
    __syncthreads();
    if (sp == 0) {
#pragma unroll
      for (int i = 0; i < K; ++i) nbr[i * kWave] = entry_idx(l[i]) < 0 ? 0 : entry_idx(l[i]);
    }
    __syncthreads();
    if (active) {
      float vq[EM];  // (read again: the merges have no registers for them)
#pragma unroll
      for (int j = 0; j < EM; ++j) vq[j] = E_T || j < E ? xs[p + j * tau] : 0.0f;
      for (int r = sp; r < K; r += S) {
        const int q = nbr[r * kWave];
        const double dq = distance(vq, q);
        D[r * kWave] = dq;
        if (a.idx) a.idx[base + r] = q;
        if (a.dist) a.dist[base + r] = static_cast<float>(dq);
      }
    }
    __syncthreads();
    double dmin = __builtin_inf();
    for (int r = 0; r < K; ++r) dmin = fmin(dmin, D[r * kWave]);
    __syncthreads();
    if (active)
      for (int r = sp; r < K; r += S) D[r * kWave] = weight(D[r * kWave], dmin);
    __syncthreads();
    if (active && (a.w || (a.mom && sp == 0))) {
      double wsum = 0.0;
      for (int r = 0; r < K; ++r) wsum += D[r * kWave];
      const double inv = 1.0 / wsum;
      if (a.w)
        for (int r = sp; r < K; r += S) a.w[base + r] = static_cast<float>(D[r * kWave] * inv);
      if (a.mom && sp == 0) {
        const int o_off = off + a.Tp;
        double yh = 0.0;
        for (int r = 0; r < K; ++r) yh += (D[r * kWave] * inv) * static_cast<double>(xs[nbr[r * kWave] + o_off]);
        mine.n = 1.0;
        mine.mo = static_cast<double>(xs[p + o_off]);
        mine.mp = yh;
      }
    }
  } else if (active) {
    // The loops over the winners stay rolled and rotate the register lists by
    // one slot per trip, so only one neighbour's coordinates are live at a time.
    int qi[K];
#pragma unroll
    for (int i = 0; i < K; ++i) qi[i] = entry_idx(l[i]);
    double D[K];  // distance, then weight, of neighbour qi[i]
    double dmin = __builtin_inf();
#pragma unroll 1
    for (int r = 0; r < K; ++r) {
      const int q = qi[0] < 0 ? 0 : qi[0];
      const double dq = distance(vp, q);
      dmin = fmin(dmin, dq);
#pragma unroll
      for (int i = 0; i < K - 1; ++i) {
        qi[i] = qi[i + 1];
        D[i] = D[i + 1];
      }
      qi[K - 1] = q;
      D[K - 1] = dq;
      if (a.idx) a.idx[base + r] = q;
      if (a.dist) a.dist[base + r] = static_cast<float>(dq);
    }
    double wsum = 0.0;
#pragma unroll 1
    for (int r = 0; r < K; ++r) {
      const double wq = weight(D[0], dmin);
      wsum += wq;
#pragma unroll
      for (int i = 0; i < K - 1; ++i) D[i] = D[i + 1];
      D[K - 1] = wq;
    }
    const double inv = 1.0 / wsum;
    if (a.w) {
#pragma unroll
      for (int i = 0; i < K; ++i) a.w[base + i] = static_cast<float>(D[i] * inv);
    }
    if (a.mom) {
      const int o_off = off + a.Tp;
      double yh = 0.0;
#pragma unroll
      for (int i = 0; i < K; ++i) yh += (D[i] * inv) * static_cast<double>(xs[qi[i] + o_off]);
      mine.n = 1.0;
      mine.mo = static_cast<double>(xs[p + o_off]);
      mine.mp = yh;
    }
  }
  if constexpr (Q >= 4) {
    if (a.mom) {  // uniform
      if (sp == 0) {
        const Mom wv = mom_wave_reduce(mine);
        if (lane == 0) wmom[qg] = wv;
      }
      __syncthreads();
      const int t4 = static_cast<int>(threadIdx.x) * 4;  // thread i merges the block of waves 4 i ..
      if (t4 < Q && blk0 + t4 * kWave < m) {
        Mom t = wmom[t4];
#pragma unroll
        for (int i = 1; i < kKnnThreads / kWave; ++i) t = mom_merge(t, wmom[t4 + i]);
        a.mom[(static_cast<int64_t>(row) * a.E_max + (E - 1)) * a.mom_blocks + blockIdx.x * (Q / 4) + threadIdx.x] = t;
      }
    }
  }
}

template <int E_T, int K, bool T1, int Q, int S, bool kQueue>
hipError_t launch_one(KnnArgs a, int nslots, int64_t L_max, hipStream_t st) {
  const void *fn = reinterpret_cast<const void *>(&k_knn<E_T, K, T1, Q, S, kQueue>);
  const size_t shm = static_cast<size_t>(scan_lds<Q, S>(K, a.lds_x, kQueue));
  if (shm > 65536) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       static_cast<int>(shm));
    if (e != hipSuccess) return e;
  }
  constexpr int kMaxY = 32768;
  const unsigned gx = static_cast<unsigned>((L_max + kWave * Q - 1) / (kWave * Q));
  for (int s0 = 0; s0 < nslots; s0 += kMaxY) {
    const int ny = nslots - s0 < kMaxY ? nslots - s0 : kMaxY;
    hipLaunchKernelGGL((k_knn<E_T, K, T1, Q, S, kQueue>), dim3(gx, static_cast<unsigned>(ny)), dim3(kWave * Q * S), shm,
                       st, a, s0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int E_T, int K, bool T1>
hipError_t launch_layout(const KnnArgs &a, int nslots, int64_t L_max, hipStream_t st) {
  constexpr bool kQ = E_T >= kQueueE;
  switch (scan_layout(nslots, L_max, E_T, K, a.mom != nullptr)) {
    case ScanLayout::kTableSplit: return launch_one<E_T, K, T1, 1, 16, kQ>(a, nslots, L_max, st);
    case ScanLayout::kSplit: return launch_one<E_T, K, T1, 4, 4, kQ>(a, nslots, L_max, st);
    case ScanLayout::kLong16:
      if constexpr (E_T <= 4) return launch_one<E_T, K, T1, 16, 1, false>(a, nslots, L_max, st);
      return hipErrorInvalidValue;  // (not chosen)
    case ScanLayout::kLong8: return launch_one<E_T, K, T1, 8, 1, false>(a, nslots, L_max, st);
    case ScanLayout::kPlainQueue:
      if constexpr (kQ) return launch_one<E_T, K, T1, 4, 1, true>(a, nslots, L_max, st);
      return hipErrorInvalidValue;  // (not chosen)
    default: return launch_one<E_T, K, T1, 4, 1, false>(a, nslots, L_max, st);
  }
}

}  // namespace
}  // namespace edm
