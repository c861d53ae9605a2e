// Batched simplex lookup with the Pearson skill computed on the fly
// (kEDM paper: Section 2.1 steps 3-4, Section 3.4 and Algorithm 3).
//
// Data layout.  A workgroup stages a tile of T targets (T in 1, 2, 4, 8, 16,
// as many as fit 160 KB of LDS for the window) over the window that its
// libraries' tables can touch, interleaved: vs[e][t] = y_t[off + e] - c_t with
// c_t the target's mean (k_target_means, one value per target and call, the
// same for every kernel), off = (E-1)*tau + Tp.
// One neighbour index q then addresses the T targets' samples as one
// contiguous LDS segment, so a wave reads them with one 128-, 64- or 32-bit
// access per lane instead of T scattered 32-bit gathers.  (The gathers' bank
// conflicts do not bound it: rows padded to T + 4 floats were 5 % slower, and
// made-up indices without any conflict took the same time.)
//
// Lane layout.  A wave walks one library's table: lane = 4 g + s, query group
// g = 0..15 handles the queries p = g, g + 16, g + 32, ... and sub-lane s the
// targets s*TPL .. s*TPL + TPL - 1 of the tile (TPL = T/4 targets per lane, at
// least 1; for T < 4 some sub-lanes idle).  Per query the four lanes of a group
// each load a quarter of the table row (K indices and weights), one query
// ahead, and pass it round by DPP; a lane gathers
// vs[q_i][targets] for i = 0..K-1 and accumulates the prediction
// yhat = sum_i w_i (y(t(q_i)+Tp) - c) with one float32 fused multiply-add per
// neighbour in index order, and the sums of the observation o = vs[p] and
// yhat: so, sp, soo, spp, sop, accumulated in float32 over runs of kRun
// queries and added to float64 totals after each run.  Both sides are taken
// relative to the target's mean (the weights sum to one, so the prediction's
// mean is near it too): the float32 runs then round values of the target's
// spread, not of its offset, and the correlation keeps errors of order 1e-8.
//
// Every pair's arithmetic is fixed: per query group the runs and the float64
// sums go over p in increasing order, then the 16 group sums meet in a
// butterfly over the lane bits of g (masks 4, 8, 16, 32).  It does not depend on T, on which
// kernel ran the pair or on how many libraries or targets shared a
// workgroup, so every kernel here and every form of the library give
// bit-identical rho.
//
// Grid kernel: blockIdx.x = tile of targets, blockIdx.y = group of 16
// library slots (one wave each); consecutive workgroups share their
// libraries' tables in L2; a wave that is done with its library loads its part
// of the next tile meanwhile.  10000 series of 2000 samples: 199 -> 166 ms for
// all E (rows loaded in quarters, tiles staged in lines: 97 -> 13 of 313 -> 240
// thousand cycles a tile at K = 8); of the rest, 75 % is the walk itself
// (issue: gathers, broadcasts and 4 fused adds a neighbour) and 19 % waiting for
// the workgroup's slowest wave.  Work-list kernel (batched plan): one item = a
// group of up to 16 libraries of similar length (longest first) against one
// tile, workgroups persistent or one per item.
#include <array>
#include <utility>

#include "../../include/edm.h"
#include "device_common.h"
#include "kernels.h"

namespace edm {
namespace {

constexpr int kGroups = 16;                  // query groups per wave
constexpr int kRun = 8;                      // queries per float32 run of the skill sums
constexpr int kXcds = 8;                     // accelerator dies (separate L2 caches) of the chip
constexpr int kTileCols = 16;                // tile columns per library group (device buckets)
constexpr int kSubs = 4;                     // lanes per query group
constexpr int kWaves = kLookupItemLibs;      // libraries per workgroup, one wave each
constexpr int kThreads = kWaves * kWave;     // 1024
// staged targets: 160 KiB less 512 bytes for the kernels' static LDS (target
// ids, offsets, the item index)
constexpr int64_t kLdsFloats = (160 * 1024 - 512) / 4;

static_assert(kGroups * kSubs == kWave, "lane layout");
static_assert(kLookupItemMaxTargets == 16, "tile layout assumes at most 16 targets");

// The lane, computed anew: what depends on it is not kept in registers across the
// tiles (items) of a workgroup, whose walk has none to spare.
__device__ __forceinline__ int own_lane() {
  int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
  asm volatile("" : "+v"(lane));
  return lane;
}

struct Sums {
  double so, sp, soo, spp, sop;
};

template <int N>
struct VecOf;
template <>
struct VecOf<1> {
  using type = float;
};
template <>
struct VecOf<2> {
  using type = float2;
};
template <>
struct VecOf<4> {
  using type = float4;
};

// A table row of K entries held by the 4 lanes of a query group: lane s loads
// kPart consecutive entries from kStart(s) on (the last parts overlap instead
// of passing the row's end), and entry i is read from its lane with a DPP
// broadcast within the quad.  (Every lane loading the whole row moves four times
// the bytes through the vector L1, 64 bytes a clock: 72 cycles a wave and query
// at K = 9 against 36 of LDS reads; and rows loaded whole one query ahead do not
// fit the registers.)
template <int K>
struct RowPart {
  static constexpr int kPart = (K + 3) / 4;
  static constexpr int start(int s) { return s * kPart < K - kPart ? s * kPart : K - kPart; }
  static constexpr int lane_of(int i) { return i / kPart; }
  static constexpr int at(int i) { return i - start(lane_of(i)); }
};
template <int S>
__device__ __forceinline__ int quad_get(int v) {
  return __builtin_amdgcn_mov_dpp(v, S * 0x55, 0xf, 0xf, false);  // quad_perm [S, S, S, S]
}
template <int S>
__device__ __forceinline__ float quad_get(float v) {
  return __int_as_float(quad_get<S>(__float_as_int(v)));
}

template <int I0, int I1, typename F>
__device__ __forceinline__ void each(F &&f) {  // f(I0), ..., f(I1 - 1) as constants
  if constexpr (I0 < I1) {
    f(std::integral_constant<int, I0>{});
    each<I0 + 1, I1>(f);
  }
}

template <int TPL>
__device__ __forceinline__ void lds_read(const float *p, float (&v)[TPL]) {
  using V = typename VecOf<TPL>::type;
  const V x = *reinterpret_cast<const V *>(p);
  if constexpr (TPL == 1) {
    v[0] = x;
  } else if constexpr (TPL == 2) {
    v[0] = x.x;
    v[1] = x.y;
  } else {
    v[0] = x.x;
    v[1] = x.y;
    v[2] = x.z;
    v[3] = x.w;
  }
}

// A library's queries split over waves: wave `part` of `parts` (a power of two)
// takes the runs part, part + parts, ... of every query group and leaves their
// float32 sums in LDS (ex: kRunSums floats a wave); after each of `rounds`
// rounds the library's first wave adds them in the order of the runs, so the
// sums are those of one wave.
struct Split {
  int part = 0, parts = 1, rounds = 0;
  float *ex = nullptr;  // of the library's first wave
};
constexpr int kRunSums = 5 * kWave;

// Skill sums of one wave's library against the staged tile (row stride T
// floats).  Lane (g, s) handles targets s*TPL + u of the tile; every lane
// returns the wave totals of its targets.  pred[u] (or null): prediction row
// of target u of the lane, written as yhat + c[u].
template <int K, int TPL, bool kPred, bool kSplit>
__device__ __forceinline__ void tile_pairs(const int32_t *__restrict__ tidx,
                                           const float *__restrict__ tw, const int m,
                                           const float *vs, const int T,
                                           float *const (&pred)[TPL], const float (&c)[TPL],
                                           Sums (&s)[TPL], const Split &split) {
  static_assert(!kSplit || TPL == 1, "exchange area: one target a lane");
  const int lane = own_lane();
  const int g = lane >> 2;
  const int sub = lane & (kSubs - 1);
  // idle sub-lanes (T < 4) read sub-lane 0's targets; their sums are unused
  const int col = sub * TPL < T ? sub * TPL : 0;
  const float *base = vs + col;
  // Row q of the tile, T (a power of two) floats apart: constant for the widths 8 and 16.
  const int lgS = TPL == 1 ? 31 - __builtin_clz(T) : (TPL == 2 ? 3 : 4);
  auto row_of = [&](int q) { return base + (static_cast<uint32_t>(q) << lgS); };
  using Row = RowPart<K>;
  const int part0 = sub * Row::kPart < K - Row::kPart ? sub * Row::kPart : K - Row::kPart;
  const int32_t *__restrict__ ti = tidx + part0;
  const float *__restrict__ tv = tw + part0;
  // The next query's part is loaded while this one's gathers run.
  int qn[Row::kPart];
  float wn[Row::kPart];
  auto load_row = [&](int p) {
    const int64_t row = static_cast<int64_t>(p) * K;
#pragma unroll
    for (int i = 0; i < Row::kPart; ++i) {
      qn[i] = ti[row + i];
      wn[i] = tv[row + i];
    }
  };
#pragma unroll
  for (int u = 0; u < TPL; ++u) s[u] = Sums{0.0, 0.0, 0.0, 0.0, 0.0};
  auto run = [&](int p0, float (&f)[TPL][5]) {
    const int pe = m < p0 + kGroups * kRun ? m : p0 + kGroups * kRun;
#pragma unroll
    for (int u = 0; u < TPL; ++u)
#pragma unroll
      for (int j = 0; j < 5; ++j) f[u][j] = 0.0f;
    for (int p = p0; p < pe; p += kGroups) {
      uint32_t qo[Row::kPart];  // LDS offset of the neighbour's row (floats)
      float w[Row::kPart];
#pragma unroll
      for (int i = 0; i < Row::kPart; ++i) {
        qo[i] = static_cast<uint32_t>(qn[i]) << lgS;
        w[i] = wn[i];
      }
      load_row(p + kGroups < m ? p + kGroups : p);
      float yh[TPL];
#pragma unroll
      for (int u = 0; u < TPL; ++u) yh[u] = 0.0f;
      float ov[TPL];
      lds_read<TPL>(row_of(p), ov);
      // gathers in chunks of kChunk neighbours (bounds the registers in flight)
      constexpr int kChunk = TPL == 4 ? (K <= 12 ? 6 : K <= 20 ? 4 : K <= 24 ? 3 : 2) : (TPL == 2 ? 8 : 16);
      each<0, (K + kChunk - 1) / kChunk>([&](auto CC) {
        constexpr int i0 = decltype(CC)::value * kChunk;
        constexpr int i1 = i0 + kChunk < K ? i0 + kChunk : K;
        float v[kChunk][TPL];
        // The chunk's gathers are issued at a raised wave priority, so the
        // SIMD's waves keep the LDS queue fed before their arithmetic.
        __builtin_amdgcn_s_setprio(1);
        each<i0, i1>([&](auto IC) {
          constexpr int i = decltype(IC)::value;
          const int o = quad_get<Row::lane_of(i)>(static_cast<int>(qo[Row::at(i)]));
          lds_read<TPL>(base + static_cast<uint32_t>(o), v[i - i0]);
        });
        __builtin_amdgcn_s_setprio(0);
        each<i0, i1>([&](auto IC) {
          constexpr int i = decltype(IC)::value;
          const float wi = quad_get<Row::lane_of(i)>(w[Row::at(i)]);
#pragma unroll
          for (int u = 0; u < TPL; ++u) yh[u] = fmaf(wi, v[i - i0][u], yh[u]);
        });
        if (K > kChunk) __builtin_amdgcn_sched_barrier(0);
      });
#pragma unroll
      for (int u = 0; u < TPL; ++u) {
        // explicit fused forms: the same operations in every instantiation
        f[u][0] += ov[u];
        f[u][1] += yh[u];
        f[u][2] = fmaf(ov[u], ov[u], f[u][2]);
        f[u][3] = fmaf(yh[u], yh[u], f[u][3]);
        f[u][4] = fmaf(ov[u], yh[u], f[u][4]);
        if constexpr (kPred) {
          if (pred[u]) pred[u][p] = yh[u] + c[u];
        }
      }
    }
  };
  auto add = [&](Sums &t, const float *f, int step) {
    t.so += static_cast<double>(f[0]);
    t.sp += static_cast<double>(f[step]);
    t.soo += static_cast<double>(f[2 * step]);
    t.spp += static_cast<double>(f[3 * step]);
    t.sop += static_cast<double>(f[4 * step]);
  };
  constexpr int kStep = kGroups * kRun;
  float f[TPL][5];
  if constexpr (kSplit) {
    float *mine = split.ex + split.part * kRunSums + lane;
    for (int r0 = 0; r0 < split.rounds * split.parts; r0 += split.parts) {
      const int p0 = g + (r0 + split.part) * kStep;
      if (p0 < m) {
        load_row(p0);
        run(p0, f);
#pragma unroll
        for (int j = 0; j < 5; ++j) mine[j * kWave] = f[0][j];
      }
      __syncthreads();
      if (split.part == 0)
        for (int w = 0; w < split.parts; ++w)
          if (g + (r0 + w) * kStep < m) add(s[0], mine + w * kRunSums, kWave);
      __syncthreads();
    }
    if (split.part != 0) return;
  } else {
    if (g < m) load_row(g);
    for (int p0 = g; p0 < m; p0 += kStep) {
      run(p0, f);
#pragma unroll
      for (int u = 0; u < TPL; ++u) add(s[u], f[u], 1);
    }
  }
#pragma unroll
  for (int u = 0; u < TPL; ++u) {
#pragma unroll
    for (int msk = kSubs; msk < kWave; msk <<= 1) {
      s[u].so += __shfl_xor(s[u].so, msk);
      s[u].sp += __shfl_xor(s[u].sp, msk);
      s[u].soo += __shfl_xor(s[u].soo, msk);
      s[u].spp += __shfl_xor(s[u].spp, msk);
      s[u].sop += __shfl_xor(s[u].sop, msk);
    }
  }
}

__device__ __forceinline__ float pair_rho(int m, const Sums &s) {
  return static_cast<float>(
      mom_rho(mom_from_shifted_sums(static_cast<double>(m), 0.0, 0.0, s.so, s.sp, s.soo, s.spp, s.sop)));
}

// A tile of T targets over the window [off, off + n), staged relative to
// cs[t] = a.cmean[target] as vs[e][t] (targets Tn..T-1 and samples past a
// target's own length zero).  A unit is 64 consecutive samples of 4 targets: a
// wave loads them as four 256-byte lines and writes one 16-byte word per lane,
// and a wave's units all belong to the same 4 targets, whose ids, lengths and
// means are wave-uniform.  The loads of a whole tile (at most 40 floats a
// thread) are in flight at once, separate from the LDS writes, so that a wave
// that is done with its library loads its share of the next tile while the
// others finish.  (Staged element by element, target fastest, a tile of 16 x
// 2000 took 97 of 313 thousand cycles.)
constexpr int kUnits = static_cast<int>((kLdsFloats + kThreads * 4 - 1) / (kThreads * 4)) + 1;
struct Tile {
  const int32_t *ids;  // the launch's target list, or nullptr: identity
  int t0, Tn;          // targets ids[t0 .. t0 + Tn)
};
template <int TQ>
struct TileLoad {
  float r[kUnits][4];
  __device__ __forceinline__ static int block_of(int j) {
    return __builtin_amdgcn_readfirstlane((static_cast<int>(threadIdx.x) / kWave + kWaves * j) / TQ);
  }
  __device__ __forceinline__ static int first_target() {  // of the wave's four
    return __builtin_amdgcn_readfirstlane((static_cast<int>(threadIdx.x) / kWave) % TQ * 4);
  }
  __device__ __forceinline__ static int id_of(const Tile &tile, int u) {
    const int t = first_target() + u < tile.Tn ? first_target() + u : 0;
    return __builtin_amdgcn_readfirstlane(tile.ids ? tile.ids[tile.t0 + t] : tile.t0 + t);
  }
  __device__ __forceinline__ void load(const LookupArgs &a, const Tile &tile, int off, int n) {
    const int lane = own_lane();
    const float *row[4];
    int last[4];  // the target's last sample: no address past it
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int id = id_of(tile, u);
      const int64_t end = off + static_cast<int64_t>(n);
      const int64_t len = a.Ly_dev && a.Ly_dev[id] < end ? a.Ly_dev[id] : (a.ldy < end ? a.ldy : end);
      row[u] = len > 0 ? a.Y + static_cast<int64_t>(id) * a.ldy : a.cmean + id;
      last[u] = len > 0 ? static_cast<int>(len) - 1 : 0;
    }
#pragma unroll
    for (int j = 0; j < kUnits; ++j) {
      const int e0 = block_of(j) * kWave;
#pragma unroll
      for (int u = 0; u < 4; ++u) r[j][u] = 0.0f;
      if (e0 >= n) continue;  // uniform
      const int i = off + e0 + lane;
#pragma unroll
      for (int u = 0; u < 4; ++u) r[j][u] = row[u][i < last[u] ? i : last[u]];  // unused where clamped
    }
  }
  __device__ __forceinline__ void store(const LookupArgs &a, const Tile &tile, int off, int n, float *vs, int T) {
    const int lane = own_lane();
    const int tq = first_target();
    float c[4];
    int end[4];  // samples of the window that the target has
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int id = id_of(tile, u);
      c[u] = a.cmean[id];
      const int64_t len = (a.Ly_dev ? a.Ly_dev[id] : a.ldy) - off;
      end[u] = tq + u < tile.Tn ? static_cast<int>(len < n ? len : n) : 0;
    }
    bool bad = false;
#pragma unroll
    for (int j = 0; j < kUnits; ++j) {
      const int e0 = block_of(j) * kWave;
      if (e0 >= n) continue;  // uniform
      const int e = e0 + lane;
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool in = e < end[u];
        bad |= in && !isfinite(r[j][u]);
        v[u] = in ? r[j][u] - c[u] : 0.0f;
      }
      if (e >= n) continue;
      float *out = vs + static_cast<int64_t>(e) * T + tq;
      if (T >= 4) {
        *reinterpret_cast<float4 *>(out) = float4{v[0], v[1], v[2], v[3]};
      } else {  // 1 or 2 targets
        out[0] = v[0];
        if (T == 2) out[1] = v[1];
      }
    }
    if (bad) atomicOr(a.status, 1);
  }
};
// Units of a tile beyond kUnits (one or two targets over a long window: the
// window outgrows the units' four targets) are staged by further rounds.
template <int TQ>
__device__ __forceinline__ void stage_rest(const LookupArgs &a, const Tile &tile, int off, int n, float *vs, int T) {
  if (TQ > 1) return;
  for (int at = kUnits * kThreads; at < n; at += kUnits * kThreads) {
    TileLoad<TQ> l;
    l.load(a, tile, off + at, n - at);
    l.store(a, tile, off + at, n - at, vs + static_cast<int64_t>(at) * T, T);
  }
}
template <int TPL>
constexpr int tile_quads() {
  return TPL;  // T = 16, 8, and 4 or fewer targets: 4, 2, 1 groups of four
}
// Ids and means of a staged tile, for the epilogues.
__device__ __forceinline__ void tile_ids(const LookupArgs &a, const Tile &tile, int T, int *tgt, float *cs) {
  const int t = static_cast<int>(threadIdx.x);
  if (t < T) {
    const int id = t < tile.Tn ? (tile.ids ? tile.ids[tile.t0 + t] : tile.t0 + t) : 0;
    tgt[t] = id;
    cs[t] = t < tile.Tn ? a.cmean[id] : 0.0f;
  }
}

// One wave's library (m queries, table tidx/tw) against the staged tile
// tgt[0..Tn): sums, then rho (and predictions) for the pairs that are
// defined (target at least as long as the library).
template <int K, int TPL, bool kSplit = false>
__device__ __forceinline__ void wave_library(const LookupArgs &a, const int32_t *tidx,
                                             const float *tw, int lib, int64_t Lx, int m,
                                             const float *vs, const float *cs, const int *tgt,
                                             int Tn, int T, const Split &split = Split{}) {
  const int lane = own_lane();
  const int sub = lane & (kSubs - 1);
  // target u of the lane, or -1 where there is none or the pair is undefined
  auto target = [&](int u) {
    const int t = sub * TPL + u;
    const bool in = sub * TPL < T && t < Tn;
    const int id = in ? tgt[t] : 0;
    return in && !(a.Ly_dev && a.Ly_dev[id] < Lx) ? id : -1;
  };
  float c[TPL];
  float *pred[TPL];
#pragma unroll
  for (int u = 0; u < TPL; ++u) {
    c[u] = 0.0f;
    pred[u] = nullptr;
  }
  Sums s[TPL];
  // predictions are written only with one target per lane (tiles of at most
  // 4 targets), which keeps the wider instantiations free of their registers
  if (TPL == 1 && a.pred) {
    const int id = target(0);
    if (id >= 0) {
      c[0] = cs[sub];
      pred[0] = a.pred + static_cast<int64_t>(id) * a.ldpred;
    }
    tile_pairs<K, TPL, TPL == 1, kSplit>(tidx, tw, m, vs, T, pred, c, s, split);
  } else {
    tile_pairs<K, TPL, false, kSplit>(tidx, tw, m, vs, T, pred, c, s, split);
  }
  if (kSplit && (split.part != 0 || m <= 0)) return;
  // (the targets are read again rather than kept over the walk, whose registers
  // they would not fit beside)
  if (a.rho && lane < kSubs) {
#pragma unroll
    for (int u = 0; u < TPL; ++u) {
      const int id = target(u);
      if (id >= 0) a.rho[static_cast<int64_t>(lib) * a.ldrho + id] = pair_rho(m, s[u]);
    }
  }
}

// Grid kernel: blockIdx.x = tile of T targets (bucket positions
// [x*T, x*T + T)), blockIdx.y = group of kWaves library slots from slot0;
// ms bounds every staged window (the dynamic LDS holds T * ms floats, and the
// split form's exchange area from ex_at on).  kSplit: 1 << lg_parts waves walk
// one library.
// kAll: one launch for every E (blockIdx.z).
template <int K, int TPL, bool kSplit, bool kAll>
__device__ __forceinline__ void lookup_block(const LookupArgs &a, int T, int nslots, int slot0, int lg_parts,
                                             int ex_at, float *vs, float *cs, int *tgt) {
  const int off = (a.E - 1) * a.tau + a.Tp;
  // targets of the launch: the host's list, or the bucket grouped on the device
  const bool dev = a.bucket_at != nullptr && a.tbl_off == nullptr;
  const int ntgt = dev ? a.bucket_at[a.E + 1] - a.bucket_at[a.E] : a.ntgt;
  const int32_t *tids = dev ? a.bucket_ids + a.bucket_at[a.E] : a.tgt_ids;
  // Host grid: blockIdx.x = tile, blockIdx.y = library group.  Device-bucket
  // grid (one dimension): workgroup i runs on XCD i % 8 (round-robin
  // dispatch); the kTileCols tile columns of a library group all go to one
  // XCD, so the workgroups an XCD runs together share two groups' tables in
  // its L2.
  int col = static_cast<int>(blockIdx.x), ncol = static_cast<int>(gridDim.x);
  int grp = static_cast<int>(blockIdx.y);
  if (dev && !kAll) {
    const int i = static_cast<int>(blockIdx.x), k = i / kXcds;
    col = k % kTileCols;
    ncol = kTileCols;
    grp = kXcds * (k / kTileCols) + i % kXcds;
  }
  const int lgp = kSplit ? lg_parts : 0;
  const int nlib = kWaves >> lgp;  // libraries of the workgroup
  const int sbase = slot0 + grp * nlib;
  int n_blk = 0;  // widest query range of the workgroup's libraries
  for (int w = 0; w < nlib; ++w) {
    const int slot = sbase + w;
    if (slot >= slot0 + nslots) break;
    const int lib = a.lib_ids ? a.lib_ids[slot] : slot;
    const int64_t Lx = a.Lx_dev ? a.Lx_dev[lib] : a.Lx_uni;
    const int mw = static_cast<int>(Lx) - off;
    n_blk = mw > n_blk ? mw : n_blk;
  }
  if (n_blk - 1 - 2 * a.excl < K) return;  // no table in this workgroup (uniform)

  const int wave = static_cast<int>(threadIdx.x) / kWave;
  const int slot = __builtin_amdgcn_readfirstlane(sbase + (wave >> lgp));
  const bool in = slot < slot0 + nslots;
  const int lib = in ? (a.lib_ids ? a.lib_ids[slot] : slot) : 0;
  const int64_t Lx = in ? (a.Lx_dev ? a.Lx_dev[lib] : a.Lx_uni) : 0;
  const int m = static_cast<int>(Lx) - off;
  const bool on = in && m - 1 - 2 * a.excl >= K;  // the table exists for this library
  const int64_t tbl = static_cast<int64_t>(slot) * a.tbl_stride;
  // tiles blockIdx.x, blockIdx.x + gridDim.x, ... (one per workgroup when the
  // host sized the grid to the target count)
  if (col * T >= ntgt) return;
  constexpr int TQ = tile_quads<TPL>();
  auto tile_at = [&](int tile) {
    const int t0 = tile * T;
    return Tile{tids, t0, ntgt - t0 < T ? ntgt - t0 : T};
  };
  TileLoad<TQ> load;
  load.load(a, tile_at(col), off, n_blk);
  for (int tile = col;;) {
    const Tile now = tile_at(tile);
    if (tile != col) __syncthreads();  // the previous tile is consumed
    tile_ids(a, now, T, tgt, cs);
    load.store(a, now, off, n_blk, vs, T);
    stage_rest<TQ>(a, now, off, n_blk, vs, T);
    __syncthreads();
    if constexpr (kSplit) {  // every wave reaches the rounds' barriers
      Split split;
      split.parts = 1 << lgp;
      split.part = wave & (split.parts - 1);
      split.rounds = (n_blk + kGroups * kRun * split.parts - 1) / (kGroups * kRun * split.parts);
      split.ex = vs + ex_at + (wave - split.part) * kRunSums;
      wave_library<K, TPL, true>(a, a.idx + tbl, a.w + tbl, lib, Lx, on ? m : 0, vs, cs, tgt, now.Tn, T, split);
    } else {
      if (on) wave_library<K, TPL>(a, a.idx + tbl, a.w + tbl, lib, Lx, m, vs, cs, tgt, now.Tn, T);
    }
    tile += ncol;
    if (tile * T >= ntgt) break;
    load.load(a, tile_at(tile), off, n_blk);
  }
}

template <int K, int TPL, bool kSplit>
__global__ __launch_bounds__(kThreads) void k_lookup(LookupArgs a, int T, int nslots, int slot0, int lg_parts,
                                                     int ex_at) {
  extern __shared__ float4 lds4[];
  __shared__ float cs[kLookupItemMaxTargets];
  __shared__ int tgt[kLookupItemMaxTargets];
  lookup_block<K, TPL, kSplit, false>(a, T, nslots, slot0, lg_parts, ex_at, reinterpret_cast<float *>(lds4), cs, tgt);
}

// The split form for every E at once (blockIdx.z = E - 1), buckets on the
// device: few series, where E_max launches of a few microseconds would find
// most buckets empty.
__global__ __launch_bounds__(kThreads) void k_lookup_all(LookupAllArgs all, int T, int nslots, int lg_parts,
                                                         int ex_at) {
  extern __shared__ float4 lds4[];
  __shared__ float cs[kLookupItemMaxTargets];
  __shared__ int tgt[kLookupItemMaxTargets];
  const int E = static_cast<int>(blockIdx.z) + 1;
  each<1, EDM_E_MAX + 1>([&](auto EC) {
    constexpr int e = decltype(EC)::value;
    if (E != e) return;
    LookupArgs a = all.a;
    a.E = e;
    a.k = e + 1;
    a.idx = all.idxE[e];
    a.w = all.wE[e];
    a.tbl_stride = all.strideE[e];
    lookup_block<e + 1, 1, true, true>(a, T, nslots, 0, lg_parts, ex_at, reinterpret_cast<float *>(lds4), cs, tgt);
  });
}

// Work-list kernel for one E (K = E + 1): persistent (counter != nullptr:
// workgroups pull items) or one workgroup per item.  An item stages a tile of
// targets once, over the window of its longest library, and wave w runs the
// item's library w against the tile.  Item fields are wave-uniform.
template <int K>
__global__ __launch_bounds__(kThreads) void k_lookup_items(LookupArgs a,
                                                            const LookupItem *__restrict__ items,
                                                            int n_items, int *counter) {
  extern __shared__ float4 lds4[];
  float *vs = reinterpret_cast<float *>(lds4);
  __shared__ float cs[kLookupItemMaxTargets];
  __shared__ int tgt[kLookupItemMaxTargets];
  __shared__ int item_s;
  const int E = K - 1;
  const int off = (E - 1) * a.tau + a.Tp;
  const int wave = static_cast<int>(threadIdx.x) / kWave;
  for (int trip = 0;; ++trip) {
    int it;
    if (counter == nullptr) {
      if (trip > 0) break;
      it = static_cast<int>(blockIdx.x);
    } else {
      __syncthreads();  // the previous item is done with vs, cs, tgt and item_s
      if (threadIdx.x == 0) item_s = atomicAdd(counter, 1);
      __syncthreads();
      it = __builtin_amdgcn_readfirstlane(item_s);
      if (it >= n_items) break;
    }
    const int at = __builtin_amdgcn_readfirstlane(items[it].lib);
    const int nlib = __builtin_amdgcn_readfirstlane(static_cast<int>(items[it].nlib));
    const int T = __builtin_amdgcn_readfirstlane(static_cast<int>(items[it].T));
    const int first = __builtin_amdgcn_readfirstlane(items[it].first);
    const int count = __builtin_amdgcn_readfirstlane(items[it].count);
    const int Tn = count < T ? count : T;
    // the first library of an item is its longest: its window covers all
    const int lib0 = __builtin_amdgcn_readfirstlane(a.item_libs[at]);
    const int ms = static_cast<int>((a.Lx_dev ? a.Lx_dev[lib0] : a.Lx_uni) - off);
    if (ms < 1) continue;  // uniform: nothing of this item can be defined
    const Tile tile{a.bucket_ids + a.bucket_at[E], first, Tn};
    tile_ids(a, tile, T, tgt, cs);
    auto stage = [&](auto QC) {
      constexpr int TQ = decltype(QC)::value;
      TileLoad<TQ> load;
      load.load(a, tile, off, ms);
      load.store(a, tile, off, ms, vs, T);
      stage_rest<TQ>(a, tile, off, ms, vs, T);
    };
    if (T >= 16) stage(std::integral_constant<int, 4>{});
    else if (T == 8) stage(std::integral_constant<int, 2>{});
    else stage(std::integral_constant<int, 1>{});
    __syncthreads();
    if (wave < nlib) {  // uniform per wave
      const int lib = __builtin_amdgcn_readfirstlane(a.item_libs[at + wave]);
      const int64_t Lx = a.Lx_dev ? a.Lx_dev[lib] : a.Lx_uni;
      const int m = static_cast<int>(Lx) - off;
      if (m - 1 - 2 * a.excl >= K) {
        const int64_t o = a.tbl_off[static_cast<int64_t>(lib) * (EDM_E_MAX + 1) + E];
        if (T >= 16)
          wave_library<K, 4>(a, a.tbl_idx + o, a.tbl_w + o, lib, Lx, m, vs, cs, tgt, Tn, T);
        else if (T == 8)
          wave_library<K, 2>(a, a.tbl_idx + o, a.tbl_w + o, lib, Lx, m, vs, cs, tgt, Tn, T);
        else
          wave_library<K, 1>(a, a.tbl_idx + o, a.tbl_w + o, lib, Lx, m, vs, cs, tgt, Tn, T);
      }
    }
  }
}

// Centring constant of every target: float32 of the float64 mean over
// [0, Ly) (Ly_dev, or L_uni for all), one wave per target summing in a fixed
// order (lane-strided, then a butterfly), so every kernel and call that
// stages the target subtracts the same value.
__global__ __launch_bounds__(256) void k_target_means(const float *__restrict__ Y, int64_t ldy,
                                                      const int64_t *__restrict__ Ly_dev, int64_t L_uni,
                                                      int64_t N, float *__restrict__ cmean) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * (256 / kWave) + threadIdx.x / kWave;
  if (t >= N) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t L = Ly_dev ? Ly_dev[t] : L_uni;
  const float *__restrict__ y = Y + t * ldy;
  double sum = 0.0;
  // (unrolled: the loads of eight steps are in flight at once)
#pragma unroll 8
  for (int64_t i = lane; i < L; i += kWave) sum += static_cast<double>(y[i]);
#pragma unroll
  for (int msk = kWave / 2; msk > 0; msk >>= 1) sum += __shfl_xor(sum, msk);
  if (lane == 0) cmean[t] = L > 0 ? static_cast<float>(sum / static_cast<double>(L)) : 0.0f;
}

using LaunchFn = hipError_t (*)(const LookupArgs &, dim3, size_t, int, int, int, int, int, hipStream_t);

template <int K, int TPL, bool kSplit>
hipError_t launch_k(const LookupArgs &a, dim3 grid, size_t shm, int T, int nslots, int slot0, int lg_parts,
                    int ex_at, hipStream_t st) {
  const void *fn = reinterpret_cast<const void *>(&k_lookup<K, TPL, kSplit>);
  if (shm > 65536) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       static_cast<int>(shm));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_lookup<K, TPL, kSplit>), grid, dim3(kThreads), shm, st, a, T, nslots, slot0, lg_parts,
                     ex_at);
  return hipGetLastError();
}

template <int TPL, bool kSplit, size_t... I>
constexpr auto make_table(std::index_sequence<I...>) {
  return std::array<LaunchFn, sizeof...(I)>{&launch_k<static_cast<int>(I) + 1, TPL, kSplit>...};
}

LaunchFn launch_fn(int k, int T, bool split) {
  constexpr auto ks = std::make_index_sequence<EDM_K_MAX>{};
  static const auto t4 = make_table<4, false>(ks);
  static const auto t2 = make_table<2, false>(ks);
  static const auto t1 = make_table<1, false>(ks);
  static const auto s1 = make_table<1, true>(ks);
  return (split ? s1 : T >= 16 ? t4 : T == 8 ? t2 : t1)[static_cast<size_t>(k - 1)];
}

// Shape of a launch: T targets a tile, 1 << lg_parts waves a library.
struct Shape {
  int T, lg_parts, ex_at;
  size_t lds;
  bool split() const { return lg_parts > 0; }
  int libs() const { return kWaves >> lg_parts; }
};

// A wave walks a library's queries one after the other, about 0.6 us a step of
// 16 queries whether it has its SIMD for itself or shares it with three others, so a launch
// of few libraries or few tiles takes one whole walk (1000 queries: 40 us) while most waves or CUs idle.
// A library's runs of 128 queries then go to 2 to 16 waves, over tiles of at
// most 4 targets: the form with the least estimated time of its workgroups in
// rounds of one per CU, a round taking (in walks) 1/W for the walk by W waves,
// three quarters of that at 4 targets, and 0.15 for staging and exchange.  One
// library of 1000 queries against 2000 targets: 48 -> 18 us with the
// predictions; eight libraries: 374 -> 331 us for sweep and cross map.
constexpr int64_t kCus = 256;
Shape shape_for(int T, int nslots, int64_t m_max, int64_t ntgt) {
  while (T > 1 && T / 2 >= ntgt) T >>= 1;  // no wider than the target count needs
  auto lds = [](int64_t floats) { return sizeof(float) * static_cast<size_t>(floats); };
  auto rounds = [&](int t, int waves) {
    const int64_t groups = (static_cast<int64_t>(nslots) * waves + kWaves - 1) / kWaves;
    return (groups * ((ntgt + t - 1) / t) + kCus - 1) / kCus;
  };
  Shape best{T, 0, 0, lds(lookup_tile_floats(T, m_max))};
  int64_t cost = rounds(T, 1) * (80 + 12);  // in 1/80 of a walk
  int Ts = T < 4 ? T : 4;
  while (Ts > 1 && lookup_tile_floats(Ts, m_max) + kWaves * kRunSums > kLdsFloats) Ts >>= 1;
  const int64_t tile = lookup_tile_floats(Ts, m_max);
  if (tile + kWaves * kRunSums > kLdsFloats) return best;
  const int64_t runs = (m_max + kGroups * kRun - 1) / (kGroups * kRun);
  for (int lg = 1; (1 << lg) <= kWaves && (1 << (lg - 1)) < runs; ++lg) {
    const int64_t c = rounds(Ts, 1 << lg) * ((60 >> lg) + 12);
    if (c >= cost) continue;
    cost = c;
    best = Shape{Ts, lg, static_cast<int>(tile), lds(tile + kWaves * kRunSums)};
  }
  return best;
}

// Workgroups of one E up to which the E go into one launch: a round of the
// chip, so that a launch of its own would not fill it.  (Sweep and cross map of E
// 1-20, one launch against one an E: 8 x 1000 219 / 345 us, 64 x 1000 912 / 976, 96 x
// 1000 1559 / 1595, 96 x 300 784 / 809; past the line 128 x 300 825 / 779.)
constexpr int64_t kAllBlocks = kCus;

}  // namespace

hipError_t launch_target_means(const float *Y, int64_t ldy, const int64_t *Ly_dev, int64_t L_uni,
                               int64_t N, float *cmean, hipStream_t st) {
  if (N <= 0) return hipSuccess;
  TimedLaunch timed(EDM_KF_LOOKUP, st);
  const int64_t blocks = (N + 3) / 4;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_target_means, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, Y, ldy, Ly_dev,
                     L_uni, N, cmean);
  return hipGetLastError();
}

int lookup_tile_targets(int64_t m) {
  int T = kLookupItemMaxTargets;
  while (T > 1 && static_cast<int64_t>(T) * m > kLdsFloats) T >>= 1;
  return T;
}

int64_t lookup_tile_floats(int T, int64_t m) { return static_cast<int64_t>(T) * m; }

hipError_t launch_lookup(const LookupArgs &a, int nslots, int64_t m_max, hipStream_t st) {
  if (nslots <= 0 || a.ntgt <= 0 || m_max <= 0) return hipSuccess;
  if (a.k < 1 || a.k > EDM_K_MAX || m_max > kLdsFloats) return hipErrorInvalidValue;
  int T = lookup_tile_targets(m_max);
  if (a.pred && T > 4) T = 4;  // the prediction-writing form
  const Shape s = shape_for(T, nslots, m_max, a.ntgt);
  const unsigned gx = static_cast<unsigned>((a.ntgt + s.T - 1) / s.T);
  const LaunchFn fn = launch_fn(a.k, s.T, s.split());
  TimedLaunch timed(EDM_KF_LOOKUP, st);
  const int max_y = 32768 * s.libs();
  for (int s0 = 0; s0 < nslots; s0 += max_y) {
    const int ns = nslots - s0 < max_y ? nslots - s0 : max_y;
    const unsigned gy = static_cast<unsigned>((ns + s.libs() - 1) / s.libs());
    hipError_t e = fn(a, dim3(gx, gy), s.lds, s.T, ns, s0, s.lg_parts, s.ex_at, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_lookup_bucket(const LookupArgs &a, int nslots, int64_t m_max, int64_t n_tgt_max,
                                hipStream_t st) {
  if (nslots <= 0 || n_tgt_max <= 0 || m_max <= 0) return hipSuccess;
  if (a.k < 1 || a.k > EDM_K_MAX || m_max > kLdsFloats || !a.bucket_at || !a.bucket_ids || a.tbl_off ||
      a.pred)
    return hipErrorInvalidValue;
  const Shape s = shape_for(lookup_tile_targets(m_max), nslots, m_max, n_tgt_max);
  // kTileCols tile columns per library group, each workgroup walking its
  // column's tiles; library groups padded to a multiple of the XCD count
  // (the kernel maps workgroups to groups XCD by XCD)
  const LaunchFn fn = launch_fn(a.k, s.T, s.split());
  TimedLaunch timed(EDM_KF_LOOKUP, st);
  const int max_slots = 65536 * s.libs();
  for (int s0 = 0; s0 < nslots; s0 += max_slots) {
    const int ns = nslots - s0 < max_slots ? nslots - s0 : max_slots;
    const int64_t groups = (ns + s.libs() - 1) / s.libs();
    const int64_t padded = (groups + kXcds - 1) / kXcds * kXcds;
    hipError_t e = fn(a, dim3(static_cast<unsigned>(padded * kTileCols), 1), s.lds, s.T, ns, s0, s.lg_parts,
                      s.ex_at, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

bool lookup_all_fits(int nslots, int64_t m_max, int64_t n_tgt_max) {
  if (nslots <= 0 || nslots > 65535 || m_max <= 0 || m_max > kLdsFloats || n_tgt_max <= 0) return false;
  const Shape s = shape_for(lookup_tile_targets(m_max), nslots, m_max, n_tgt_max);
  return s.split() && (nslots + s.libs() - 1) / s.libs() * ((n_tgt_max + s.T - 1) / s.T) <= kAllBlocks;
}

hipError_t launch_lookup_all(const LookupAllArgs &all, int E_max, int nslots, int64_t m_max, int64_t n_tgt_max,
                             hipStream_t st) {
  if (!lookup_all_fits(nslots, m_max, n_tgt_max) || E_max < 1 || E_max > EDM_E_MAX || !all.a.bucket_at ||
      !all.a.bucket_ids || all.a.tbl_off || all.a.pred)
    return hipErrorInvalidValue;
  const Shape s = shape_for(lookup_tile_targets(m_max), nslots, m_max, n_tgt_max);
  if (s.lds > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_lookup_all),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(s.lds));
    if (e != hipSuccess) return e;
  }
  TimedLaunch timed(EDM_KF_LOOKUP, st);
  const dim3 grid(static_cast<unsigned>((n_tgt_max + s.T - 1) / s.T),
                  static_cast<unsigned>((nslots + s.libs() - 1) / s.libs()), static_cast<unsigned>(E_max));
  hipLaunchKernelGGL(k_lookup_all, grid, dim3(kThreads), s.lds, st, all, s.T, nslots, s.lg_parts, s.ex_at);
  return hipGetLastError();
}

hipError_t launch_lookup_items(const LookupArgs &a, int E, const LookupItem *items, int n_items,
                               int *counter, int64_t lds_floats, int wg_per_cu, int n_cu,
                               hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  using Fn = void (*)(LookupArgs, const LookupItem *, int, int *);
#define EDM_FN(E) &k_lookup_items<E + 1>
  static const Fn fns[EDM_E_MAX] = {EDM_FN(1),  EDM_FN(2),  EDM_FN(3),  EDM_FN(4),  EDM_FN(5),
                                    EDM_FN(6),  EDM_FN(7),  EDM_FN(8),  EDM_FN(9),  EDM_FN(10),
                                    EDM_FN(11), EDM_FN(12), EDM_FN(13), EDM_FN(14), EDM_FN(15),
                                    EDM_FN(16), EDM_FN(17), EDM_FN(18), EDM_FN(19), EDM_FN(20)};
#undef EDM_FN
  if (E < 1 || E > EDM_E_MAX || lds_floats > kLdsFloats) return hipErrorInvalidValue;
  const size_t shm = static_cast<size_t>(lds_floats) * sizeof(float);
  const void *fn = reinterpret_cast<const void *>(fns[E - 1]);
  if (shm > 65536) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       static_cast<int>(shm));
    if (e != hipSuccess) return e;
  }
  TimedLaunch timed(EDM_KF_LOOKUP, st);
  if (wg_per_cu <= 0) {
    hipLaunchKernelGGL(fns[E - 1], dim3(static_cast<unsigned>(n_items)), dim3(kThreads), shm,
                       st, a, items, n_items, static_cast<int *>(nullptr));
  } else {
    int grid = wg_per_cu * n_cu;
    if (grid > n_items) grid = n_items;
    hipLaunchKernelGGL(fns[E - 1], dim3(static_cast<unsigned>(grid)), dim3(kThreads), shm, st,
                       a, items, n_items, counter);
  }
  return hipGetLastError();
}

}  // namespace edm
