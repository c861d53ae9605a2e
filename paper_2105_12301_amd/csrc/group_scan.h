// Exact scan of a group of embedding dimensions (sweep_multi.hip says how one
// candidate scan serves several E), as a device function.
#pragma once

#include "../../include/edm.h"
#include "device_common.h"
#include "kernels.h"
#include "scan_common.h"

#pragma clang fp contract(off)

namespace edm {
namespace {

constexpr int kPendQ = 16;  // queue positions per lane of a group's scan

// LDS of a group's queues and merges, beyond the staged series.
template <int ELO, int EHI, int Q, int S, bool kQueue>
constexpr size_t group_extra_lds() {
  const size_t queue =
      kQueue ? (ELO == EHI ? kPendBytes : sizeof(int32_t) * kPendQ * kWave) * static_cast<size_t>(Q * S) : 0;
  const size_t merge = merge_bytes<Q, S>(EHI + 1);
  return queue > merge ? queue : merge;
}

// One workgroup's share of a batched scan: query block `bx` of row `row`,
// every E in [ELO, EHI].  Called by the grid kernel and by the persistent
// kernel; every early return is uniform across the workgroup.  kQueue: improving
// candidates are queued, otherwise inserted as they come.  kGate: queued insertions
// skip the lists that the row does not need.
template <int ELO, int EHI, int Q, int S, bool kQueue, bool kGate = false>
__device__ __forceinline__ void group_scan(const KnnArgs &a, const int row, const int bx,
                                           float *__restrict__ smem) {
  constexpr int kT = kWave * Q * S;
  constexpr int NG = EHI - ELO + 1;
  constexpr int TOT = list_off<ELO>(EHI + 1);
  __shared__ Mom wmom[Q][NG];
  const uint32_t need = a.need_dev ? a.need_dev[row] : a.need;
  const float *__restrict__ x = a.X + static_cast<int64_t>(row) * a.ldx;
  const int L = static_cast<int>(a.L_dev ? a.L_dev[row] : a.L_uni);
  const int Tp = a.Tp;
  constexpr uint32_t kOfGroup = ((1u << EHI) - 1u) & ~((1u << (ELO - 1)) - 1u);
  if (a.mom == nullptr ? (need & kOfGroup) == 0u : ELO > a.E_max) return;  // no list of the group is wanted
  // m(E) = queries = candidates at dimension E (tau = 1)
  const int m_lo = L - (ELO - 1) - Tp;
  const int m_hi = L - (EHI - 1) - Tp;
  if (m_lo - 1 < ELO + 1) return;  // no E of the group is feasible
  const int blk0 = bx * (kWave * Q);
  if (blk0 >= m_lo) return;

  const float *xs = stage_scan<kT>(x, L, smem, a.status);

  const int lane = threadIdx.x & (kWave - 1);
  // wave-uniform: readfirstlane lets the compiler keep them (and the self step) scalar
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int qg = wave % Q, sp = wave / Q;
  const int p0 = blk0 + qg * kWave;
  const int p = p0 + lane;

  float vp[EHI];
#pragma unroll
  for (int j = 0; j < EHI; ++j) vp[j] = (p < m_lo && p + j < L) ? xs[p + j] : 0.0f;

  double l[TOT];
  static_for<ELO, EHI>([&](auto EC) {
    constexpr int E = decltype(EC)::value;
    constexpr int OFF = list_off<ELO>(E);
    // lists of E that are not wanted stay idle (kth = -1)
    const bool act = p < L - (E - 1) - Tp && E <= a.E_max && (a.mom != nullptr || ((need >> (E - 1)) & 1u));
#pragma unroll
    for (int i = 0; i < E + 1; ++i) l[OFF + i] = act ? entry_empty() : entry_idle();
  });

  // steps s = -(kWave - 1) .. m_lo - 1; split sp takes one contiguous share
  const int share = (m_lo + kWave - 1 + S - 1) / S;
  const int s0 = -(kWave - 1) + sp * share;
  const int s_end = s0 + share < m_lo ? s0 + share : m_lo;
  // every lane's q < m_hi: valid for all E
  const int s_full = m_hi - (kWave - 1) < s_end ? m_hi - (kWave - 1) : s_end;
  double *const extra = reinterpret_cast<double *>(smem + a.lds_x);
  if constexpr (!kQueue) {
    if (p0 < m_lo)
      scan_steps<ELO, EHI, true, kScanUnroll>(
          vp, xs, lane, 1, s0, s_end, s_full,
          [&](int s, int q, const float(&key)[NG], auto edge) {
            if (s == p0) return;  // (wave-uniform)
            constexpr bool kEdge = decltype(edge)::value;
            float d[NG];  // negative: the key improves E's list (see below)
            static_for<ELO, EHI>([&](auto EC) {
              constexpr int E = decltype(EC)::value;
              d[E - ELO] = key[E - ELO] - entry_key(l[list_off<ELO>(E) + E]);
              if constexpr (kEdge)
                if (s >= s_end || q < 0 || q >= L - (E - 1) - Tp) d[E - ELO] = 0.0f;
            });
            float any = d[0];
#pragma unroll
            for (int g = 1; g < NG; ++g) any = fminf(any, d[g]);
            if (__builtin_amdgcn_ballot_w64(any < 0.0f) == 0) return;
            static_for<ELO, EHI>([&](auto EC) {
              constexpr int E = decltype(EC)::value;
              const bool want = d[E - ELO] < 0.0f;
              if (NG == 1 || __builtin_amdgcn_ballot_w64(want))
                list_insert<list_off<ELO>(E), E + 1, TOT>(
                    l, entry(want ? key[E - ELO] : __builtin_inff(), q < 0 ? 0 : q));
            });
          },
          []() {});
  } else if constexpr (NG == 1) {
    // one E: its improving entries are queued with their keys
    Pending pend(extra);
    auto flush = [&]() { pend.drain([&](double e) { list_insert<0, ELO + 1, TOT>(l, e); }); };
    if (p0 < m_lo) {
      scan_steps<ELO, EHI, true, kPendStep>(
          vp, xs, lane, 1, s0, s_end, s_full,
          [&](int s, int q, const float(&key)[NG], auto edge) {
            const bool in = !decltype(edge)::value || (s < s_end && static_cast<unsigned>(q) < static_cast<unsigned>(m_lo));
            pend.push(entry(key[0], q), in && s != p0 && key[0] < entry_key(l[ELO]));
          },
          [&]() {
            if (pend.full()) flush();
          });
      flush();
    }
  } else if (p0 < m_lo) {
    // Candidates that improve some list of the group are queued (their index
    // alone) and inserted in batches, with every E's key recomputed.
    int32_t *pend = reinterpret_cast<int32_t *>(extra) + wave * (kPendQ * kWave) + lane;
    int n_pend = 0;
    [[maybe_unused]] const uint32_t needed = __builtin_amdgcn_readfirstlane(static_cast<int>(need));
    // (Every list of the group, wanted or not: their insertions are independent
    // instructions of one block.  Skipping unwanted ones by a branch each (kGate)
    // costs 5-24 % where all are wanted, and both loops in one kernel spill.)
    auto flush = [&]() {
#pragma unroll 1
      for (int i = 0; i < kPendQ; ++i) {
        const bool has = i < n_pend;
        if (__builtin_amdgcn_ballot_w64(has) == 0) break;
        const int q = has ? pend[i * kWave] : 0;
        float acc = 0.0f;
        static_for<0, EHI - 1>([&](auto JC) {
          constexpr int j = decltype(JC)::value;
          const float d = vp[j] - xs[q + j];
          acc = acc + d * d;
          if constexpr (j + 1 >= ELO) {
            constexpr int E = j + 1;
            if constexpr (kGate)
              if (!((needed >> (E - 1)) & 1u)) return;
            const float key = has && q < L - (E - 1) - Tp ? acc : __builtin_inff();
            list_insert<list_off<ELO>(E), E + 1, TOT>(l, entry(key, q));
          }
        });
      }
      n_pend = 0;
    };
    scan_steps<ELO, EHI, true, kScanUnroll>(
        vp, xs, lane, 1, s0, s_end, s_full,
        [&](int s, int q, const float(&key)[NG], auto edge) {
          // Sign bit set: the candidate's key improves E's list (the sign of
          // the float32 difference of finite keys is exact; an empty list,
          // kth = +inf, gives -inf and an idle one, kth = -1, a positive value).
          uint32_t any = 0;
          static_for<ELO, EHI>([&](auto EC) {
            constexpr int E = decltype(EC)::value;
            const uint32_t b = __float_as_uint(key[E - ELO] - entry_key(l[list_off<ELO>(E) + E]));
            any |= !decltype(edge)::value || q < L - (E - 1) - Tp ? b : 0u;
          });
          const bool in = !decltype(edge)::value || (s < s_end && q >= 0);
          if (in && s != p0 && static_cast<int32_t>(any) < 0) {
            pend[n_pend * kWave] = q;
            ++n_pend;
          }
        },
        [&]() {
          if (__builtin_amdgcn_ballot_w64(n_pend > kPendQ - kScanUnroll)) flush();
        });
    flush();
  }
  if constexpr (S > 1) {  // (the queues are drained: their LDS serves the merges)
    static_for<ELO, EHI>([&](auto EC) {
      constexpr int E = decltype(EC)::value;
      merge_splits<Q, S, list_off<ELO>(E), E + 1, TOT>(l, extra);
    });
  }

  // Epilogue per E: float64 distances and weights of the winners, the
  // self-prediction Tp ahead, and the block's co-moments.
  static_for<ELO, EHI>([&](auto EC) {
    constexpr int E = decltype(EC)::value;
    int qi[E + 1];
#pragma unroll
    for (int i = 0; i < E + 1; ++i) qi[i] = entry_idx(l[list_off<ELO>(E) + i]);
    if (S == 1 || sp == 0) {
      const Mom mine = finish_list<E, EHI>(a, row, p, L, Tp, need, vp, qi, xs);
      if (a.mom) {  // uniform
        const Mom wv = mom_wave_reduce(mine);
        if (lane == 0) wmom[qg][E - ELO] = wv;
      }
    }
  });
  if (a.mom == nullptr) return;
  __syncthreads();
  // one thread per block of 256 queries and E
  if (static_cast<int>(threadIdx.x) < NG * (Q / 4)) {
    const int g = static_cast<int>(threadIdx.x) % NG, blk = static_cast<int>(threadIdx.x) / NG;
    const int E = ELO + g;
    const int mE = L - (E - 1) - Tp;
    if (E <= a.E_max && mE - 1 >= E + 1 && blk0 + blk * kKnnThreads < mE) {
      Mom t = wmom[4 * blk][g];
#pragma unroll
      for (int w = 1; w < 4; ++w) t = mom_merge(t, wmom[4 * blk + w][g]);
      a.mom[(static_cast<int64_t>(row) * a.E_max + (E - 1)) * a.mom_blocks + bx * (Q / 4) + blk] = t;
    }
  }
}

}  // namespace
}  // namespace edm
