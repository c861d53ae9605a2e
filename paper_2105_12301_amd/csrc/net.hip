// Learned embedding-dimension surrogate: kernels for training (float32) and
// inference of a small 1-D convolutional network.
//
// The network (labels come from the simplex E sweep, the method's own E
// selection of Section 2.1 step 1 / Section 3.4 of the kEDM paper):
//   x[L] -> conv(1->C, KW) -> ReLU -> conv(C->C, KW) -> ReLU -> conv(C->C, KW)
//        -> ReLU -> mean over time -> linear(C->20) -> logits over E = 1..20
// with zero "same" padding.
//
// Training (float32): activations and their gradients are [B][L][C] in the
// workspace, channels fastest.  The C -> C convolutions, their data gradients
// (the same contraction with the weights transposed and flipped) and their
// weight gradients run on v_mfma_f32_32x32x2_f32: float32 operands, float32
// accumulation.  Weight gradients reduce over (series, time) in slices with a
// second pass over the slices, so no float atomics are involved and results
// are deterministic.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/edm.h"
#include "net_kernels.h"

namespace edm {
namespace {

constexpr int KW = EDM_NET_KW;
constexpr int HALO = KW / 2;
constexpr int NCLS = EDM_NET_CLASSES;

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kMaxC = EDM_NET_C_MAX;
__host__ __device__ constexpr int pad32(int C) { return (C + 31) / 32 * 32; }
// Blocks of 8 input channels that the products of a C -> C layer run over, and
// the channels that a workgroup's threads are dealt out over (a power of two).
__host__ __device__ constexpr int blocks8(int C) { return (C + 7) / 8; }
__host__ __device__ constexpr int lg_lanes(int C) { return C <= 8 ? 3 : (C <= 16 ? 4 : (C <= 32 ? 5 : 6)); }

// The contraction of a C -> C layer runs over e = 7 ci + k in ascending order
// (channels, then taps), two at a time: v_mfma_f32_32x32x2_f32 adds its two
// products one after the other with a rounding each, as two fused
// multiply-adds, so every output is the same chain of fused multiply-adds that a
// vector kernel walking the channels and taps in order computes.
//
// Weights in fragment order: element q of wf[u][cot][lane] (float4) holds
// A[co = 32 cot + lane % 32][e = 2 (4 u + q) + lane / 32], A[co][7 ci + k] =
// w[co][ci][k], or with `flip` w[ci][co][KW - 1 - k]; zero outside C.  Matrices
// of a pass: layers 2 and 3, then (a training pass) layers 3 and 2 flipped.
__host__ __device__ constexpr int frag_floats(int C) { return KW * 8 * blocks8(C) * pad32(C); }
__device__ __forceinline__ void weight_frag(const float *__restrict__ w2, const float *__restrict__ w3, int C, int el,
                                            float *__restrict__ wf) {
  const int n_cot = pad32(C) / 32;
  const int at = el / frag_floats(C), i = el - at * frag_floats(C);
  const bool flip = at >= 2;
  const float *__restrict__ w = at == 0 || at == 3 ? w2 : w3;
  const int q = i & 3, lane = (i >> 2) & 63, cot = (i >> 8) % n_cot, u = (i >> 8) / n_cot;
  const int e = 2 * (4 * u + q) + (lane >> 5);
  const int co = 32 * cot + (lane & 31), ci = e / KW, k = e % KW;
  float v = 0.0f;
  if (co < C && ci < C) v = flip ? w[(ci * C + co) * KW + (KW - 1 - k)] : w[(co * C + ci) * KW + k];
  wf[el] = v;
}

// Layer 1: y[b][t][c] = relu(sum_k w[c][k] x[b][t + k - HALO] + bias[c]).
// Bound by its output's HBM writes; a thread holds its channel's weights.
// Workgroup i: time tile i % tiles of series i / tiles, and from B * tiles on
// 256 of the layers' weights in fragment order (a launch of their own was
// 5 of 34 us where one short series passes a small network).
constexpr int T1 = 128;  // time steps per workgroup
__global__ __launch_bounds__(256) void k_conv1(const float *__restrict__ x, int64_t ldx, int B, int C, int L,
                                               const float *__restrict__ w, const float *__restrict__ bias,
                                               float *__restrict__ y, const float *__restrict__ w2,
                                               const float *__restrict__ w3, float *__restrict__ wf) {
  __shared__ float xs[T1 + KW - 1];
  const int tid = threadIdx.x, tiles = (L + T1 - 1) / T1;
  const int64_t wg = static_cast<int64_t>(blockIdx.x);
  if (wg >= static_cast<int64_t>(B) * tiles) {
    weight_frag(w2, w3, C, static_cast<int>(wg - static_cast<int64_t>(B) * tiles) * 256 + tid, wf);
    return;
  }
  const int b = static_cast<int>(wg / tiles), t0 = static_cast<int>(wg % tiles) * T1;
  for (int i = tid; i < T1 + KW - 1; i += 256) {
    const int t = t0 + i - HALO;
    xs[i] = t >= 0 && t < L ? x[static_cast<int64_t>(b) * ldx + t] : 0.0f;
  }
  __syncthreads();
  const int c = tid & 63;
  if (c >= C) return;
  float wr[KW];
#pragma unroll
  for (int k = 0; k < KW; ++k) wr[k] = w[c * KW + k];
  const float bc = bias[c];
  float *out = y + (static_cast<int64_t>(b) * L + t0) * C + c;
  const int n = L - t0 < T1 ? L - t0 : T1;
#pragma unroll 4
  for (int t = tid >> 6; t < n; t += 4) {
    float s = 0.0f;
#pragma unroll
    for (int k = 0; k < KW; ++k) s = fmaf(wr[k], xs[t + k], s);
    out[static_cast<int64_t>(t) * C] = fmaxf(s + bc, 0.0f);
  }
}

// C -> C convolution over time, x, y [B][L][C]:
//   kBack = false: y = relu(conv(x) + bias)
//   kBack = true:  y = conv(x) where aprev > 0, else 0
// kMask: the input is x > 0 ? chan[b][c] : 0 (the pooled layer's gradient,
// which is one value per channel on the layer's support; never stored).
//
// A workgroup (4 waves) computes CR time steps; the input window sits in LDS
// [t][channel] (odd row stride: a wave's 32 rows fall on distinct banks), every
// wave owns two time tiles and all output-channel tiles.  Per step one LDS
// word per time tile and a quarter of a 16-byte load per channel tile (weights
// from L2, one block of 8 channels ahead) feed 2 x 2 products of 64 cycles, so
// the matrix cores bound it: 22 GFLOP at C = 64, 256 x 1500, whose vector form
// took 0.45-0.49 ms.  Only the blocks of 8 that hold input channels are staged
// and multiplied (products of zeros change no bit).
constexpr int CR = 256;
template <int NCO, bool kBack, bool kMask>
__global__ __launch_bounds__(256, 2) void k_conv_f32(const float *__restrict__ x, const float *__restrict__ chan, int C,
                                                  int L, const f32x4_t *__restrict__ wf,
                                                  const float *__restrict__ bias, const float *__restrict__ aprev,
                                                  float *__restrict__ y) {
  constexpr int CP = 32 * NCO, XS = CP + 1;
  extern __shared__ __attribute__((aligned(16))) float conv_lds[];
  const int b = blockIdx.y, t0 = blockIdx.x * CR, tid = threadIdx.x;
  const float *xb = x + static_cast<int64_t>(b) * L * C;
  // Staging: a thread's channel is fixed; eight clamped loads are in flight at
  // once, and what lies outside the series or the channels becomes zero after.
  {
    constexpr int kBatch = 8;
    // rows that some lane of a working wave uses: its 64 time steps and the halo
    const int rows = (L - t0 < CR ? (L - t0 + 63) / 64 * 64 : CR) + KW - 1;
    const int lgc = lg_lanes(C), RP = 256 >> lgc;  // rows per round of the workgroup
    const int c = tid & ((1 << lgc) - 1);
    const bool has = c < C;
    const float *xc = xb + (has ? c : 0);
    const float ch = kMask && has ? chan[b * C + c] : 0.0f;
#pragma unroll 1
    for (int r0 = tid >> lgc; r0 < rows; r0 += RP * kBatch) {
      float v[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int t = t0 + r0 + RP * i - HALO;
        v[i] = xc[static_cast<int64_t>(t < 0 ? 0 : (t < L ? t : L - 1)) * C];
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int r = r0 + RP * i, t = t0 + r - HALO;
        float w = v[i];
        if constexpr (kMask) w = w > 0.0f ? ch : 0.0f;
        if (r < rows) conv_lds[r * XS + c] = has && t >= 0 && t < L ? w : 0.0f;
      }
    }
  }
  __syncthreads();
  const int wave = tid >> 6, lane = tid & 63, n = lane & 31, h = lane >> 5;
  if (t0 + 64 * wave >= L) return;
  f32x16_t acc[2][NCO];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int c = 0; c < NCO; ++c) acc[j][c] = f32x16_t{};
  const f32x4_t *wl = wf + lane;
  constexpr int kQ = KW;  // float4 rounds of a block of 8 channels: 56 products' pairs / 2 / 4
  // lane's LDS word of step s of a block: e = 2 s + h, row n + k, channel e / 7
  const float *xr[KW];
#pragma unroll
  for (int s = 0; s < KW; ++s) {
    const int e = 2 * s + h;
    xr[s] = conv_lds + (64 * wave + n + e % KW) * XS + e / KW;
  }
  f32x4_t av[kQ][NCO];
#pragma unroll
  for (int u = 0; u < kQ; ++u)
#pragma unroll
    for (int c = 0; c < NCO; ++c) av[u][c] = wl[(u * NCO + c) * 64];
#pragma unroll 1
  for (int blk = 0, n_blk = blocks8(C); blk < n_blk; ++blk) {
    const int nb = blk + 1 < n_blk ? blk + 1 : blk;
    f32x4_t an[kQ][NCO];
#pragma unroll
    for (int u = 0; u < kQ; ++u)
#pragma unroll
      for (int c = 0; c < NCO; ++c) an[u][c] = wl[((nb * kQ + u) * NCO + c) * 64];
#pragma unroll
    for (int s = 0; s < 4 * kQ; ++s) {
      float bv[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) bv[j] = xr[s % KW][32 * j * XS + 2 * (s / KW)];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int c = 0; c < NCO; ++c)
          acc[j][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s / 4][c][s % 4], bv[j], acc[j][c], 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < KW; ++s) xr[s] += 8;
#pragma unroll
    for (int u = 0; u < kQ; ++u)
#pragma unroll
      for (int c = 0; c < NCO; ++c) av[u][c] = an[u][c];
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int t = t0 + 64 * wave + 32 * j + n;
    if (t >= L) continue;
    const int64_t at = (static_cast<int64_t>(b) * L + t) * C;
#pragma unroll
    for (int c = 0; c < NCO; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int co = 32 * c + 8 * q + 4 * h;
        if (co >= C) continue;
        // four channels at a time where they are one aligned word of 16 bytes
        if ((C & 3) == 0) {
          f32x4_t v;
          f32x4_t m = {1.0f, 1.0f, 1.0f, 1.0f};
          if constexpr (kBack) m = *reinterpret_cast<const f32x4_t *>(aprev + at + co);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            v[u] = acc[j][c][4 * q + u];
            if constexpr (kBack) v[u] = m[u] > 0.0f ? v[u] : 0.0f;
            else v[u] = fmaxf(v[u] + bias[co + u], 0.0f);
          }
          *reinterpret_cast<f32x4_t *>(y + at + co) = v;
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (co + u >= C) continue;
            float v = acc[j][c][4 * q + u];
            if constexpr (kBack) v = aprev[at + co + u] > 0.0f ? v : 0.0f;
            else v = fmaxf(v + bias[co + u], 0.0f);
            y[at + co + u] = v;
          }
        }
      }
  }
}

// ---- BF16 inference form (matrix cores) ------------------------------------
// One kernel runs the whole stack on a tile of time steps; no activation
// leaves the compute unit.  (Three convolution kernels with float32
// activations in HBM moved 2.4 GB for 1024 series of 1500 samples, C = 64, and
// took 2.39 ms; this form takes 0.28 ms, 0.1 of it matrix-core time.)
//
// The contraction over (tap k, input channel i) runs on
// v_mfma_f32_32x32x16_bf16: A = weights [co][k*C + i], B = the input window
// [k*C + i][t] = x[i][t + k - HALO], both BF16, FP32 accumulation.  Activations
// live in LDS transposed to [t][channel], so every lane's eight K values
// (eight consecutive channels at one tap) are one aligned 16-byte read; rows
// are padded by 16 bytes against bank conflicts.  Layer 1 (one input channel)
// is float32 FMAs; each layer's output is rounded to BF16 as the next layer's
// input.
//
// A workgroup (8 waves, two a SIMD: one's products hide the other's reads and
// rounding) computes TO time steps of layer 3: 256 rows of layer 2 (3 more on
// either side) from 262 of layer 1.  Every wave owns one time tile and every
// output-channel tile.  160 KB of LDS hold one layer's weights beside the two
// activation tiles, so the weights alternate: the next layer's are loaded into
// registers while this layer's products run.  Layer 3's outputs are summed
// over time in registers; k_pool_parts adds the workgroups' sums of a series
// in order and applies the linear layer.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int TR = 256;            // rows of layers 2 and 3 per tile
constexpr int TO = TR - 2 * HALO;  // time steps finished per tile
constexpr int R1 = TR + 2 * HALO;  // rows of layer 1
constexpr int IT = 512;            // threads of a workgroup
constexpr int kInferWgs = 512;     // workgroups wanted: a series' tiles are split until then

__device__ __forceinline__ uint16_t to_bf16(float f) {  // round to nearest even (finite f)
  const uint32_t u = __float_as_uint(f);
  return static_cast<uint16_t>((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return static_cast<uint32_t>(to_bf16(lo)) | (static_cast<uint32_t>(to_bf16(hi)) << 16);
}

template <int C>
struct Infer {
  static constexpr int XS = C + 8;       // row stride of the activations (BF16 values)
  static constexpr int WS = KW * C + 8;  // row stride of the weights
  static constexpr int NCO = C / 32, NCC = C / 16;
  static constexpr int NPF = (C * WS / 8 + IT - 1) / IT;  // 16-byte words of a layer's weights per thread
  static constexpr int NW = NPF * IT;                   // ... padded to whole rounds of the workgroup
  static constexpr int kA2 = R1 * XS, kW = 2 * R1 * XS, kX = kW + NW * 8;  // LDS offsets (BF16 values)
  static constexpr size_t lds = sizeof(uint16_t) * kX + sizeof(float) * (R1 + 2 * HALO);
};

// w[co][ci][k] float32 -> wb[co][k][ci] BF16 of two layers, `words` 16-byte
// words each: rows of KW*C + 8 values, padding zero.
__global__ void k_w_to_bf16(const float *__restrict__ w2, const float *__restrict__ w3, int C, int words,
                            uint16_t *__restrict__ wb) {
  const int WS = KW * C + 8;
  const int i = static_cast<int>(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= 2 * words * 8) return;
  const float *w = i < words * 8 ? w2 : w3;
  const int e = i < words * 8 ? i : i - words * 8;
  const int co = e / WS, r = e - co * WS;
  const int k = r / C, ci = r - k * C;
  wb[i] = co < C && r < KW * C ? to_bf16(w[(co * C + ci) * KW + k]) : static_cast<uint16_t>(0);
}

// Sums over time of layer 3: part[b][split][C], split = blockIdx.x of gridDim.x.
// kShort: the series ends well before its only tile, and waves without a row of
// it skip their products (4000 series of 8, C = 32: 147 -> 76 us with two
// workgroups a CU; beside whole tiles the branches cost 0.5 %).
template <int C, bool kShort>
__global__ __launch_bounds__(IT, C == 32 ? 4 : 2) void k_net_infer(const float *__restrict__ X, int64_t ldx, int L,
                                                   const float *__restrict__ w1, const float *__restrict__ b1,
                                                   const float *__restrict__ b2, const float *__restrict__ b3,
                                                   const u32x4_t *__restrict__ wb, int tiles,
                                                   float *__restrict__ part) {
  using I = Infer<C>;
  static_assert(C % 32 == 0 && C <= 64, "C must be 32 or 64");
  extern __shared__ __attribute__((aligned(16))) uint16_t lds_bf16[];
  uint16_t *a1 = lds_bf16, *a2 = lds_bf16 + I::kA2, *ws = lds_bf16 + I::kW;
  float *xin = reinterpret_cast<float *>(lds_bf16 + I::kX);
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *x = X + static_cast<int64_t>(blockIdx.y) * ldx;

  u32x4_t pf[I::NPF];
  auto load_w = [&](int layer) {  // the weights of layer 2 (0) or 3 (1) into registers
#pragma unroll
    for (int i = 0; i < I::NPF; ++i) pf[i] = wb[layer * I::NW + tid + IT * i];
  };
  auto store_w = [&]() {
#pragma unroll
    for (int i = 0; i < I::NPF; ++i) reinterpret_cast<u32x4_t *>(ws)[tid + IT * i] = pf[i];
  };
  // layer 1: a thread's CH channels c0.. at times tid / CG + ... (C = 32: four,
  // so that two workgroups share a CU in 128 registers without spills)
  constexpr int CH = C == 32 ? 4 : 8, CG = C / CH;
  const int c0 = (tid % CG) * CH;
  float w1r[CH][KW], b1r[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    b1r[c] = b1[c0 + c];
#pragma unroll
    for (int k = 0; k < KW; ++k) w1r[c][k] = w1[(c0 + c) * KW + k];
  }
  // products of 256 rows of `in` (row 32 wave + n of this lane) with the staged weights
  const int row = 32 * wave + n;
  f32x16_t acc[I::NCO];
  auto conv = [&](const uint16_t *in) {
#pragma unroll
    for (int c = 0; c < I::NCO; ++c) acc[c] = f32x16_t{};
#pragma unroll
    for (int k = 0; k < KW; ++k) {
#pragma unroll
      for (int cc = 0; cc < I::NCC; ++cc) {
        bf16x8_t aop[I::NCO];
        const bf16x8_t bop = *reinterpret_cast<const bf16x8_t *>(in + (row + k) * I::XS + 16 * cc + 8 * h);
#pragma unroll
        for (int c = 0; c < I::NCO; ++c)
          aop[c] = *reinterpret_cast<const bf16x8_t *>(ws + (32 * c + n) * I::WS + k * C + 16 * cc + 8 * h);
#pragma unroll
        for (int c = 0; c < I::NCO; ++c)
          acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aop[c], bop, acc[c], 0, 0, 0);
      }
    }
  };
  float sum[I::NCO][16];  // this lane's column sums: channel 32 c + 8 (v >> 2) + 4 h + (v & 3)
#pragma unroll
  for (int c = 0; c < I::NCO; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[c][v] = 0.0f;
  auto bias = [&](const float *b, int c, int v) { return b[32 * c + 8 * (v >> 2) + 4 * h + (v & 3)]; };

  load_w(0);
  // rows 256 .. 261 of layer 2 only feed discarded time steps; they stay zero
  for (int i = tid; i < 2 * HALO * I::XS; i += IT) a2[TR * I::XS + i] = 0;
#pragma unroll 1
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int t0 = tile * TO;
    const int rows = L - t0 < TO ? L - t0 : TO;  // of layer 3 that lie in the series
    // xin[i] = x[t0 - 3 HALO + i], zero outside the series
    for (int i = tid; i < R1 + 2 * HALO; i += IT) {
      const int t = t0 - 3 * HALO + i;
      xin[i] = t >= 0 && t < L ? x[t] : 0.0f;
    }
    __syncthreads();  // (also: the previous tile's layer 3 is done with the weights)
    store_w();
    load_w(1);
    // layer 1: row r is time t0 - 2 HALO + r
    for (int r = tid / CG; r < (kShort ? rows + 4 * HALO : R1); r += IT / CG) {
      const int t = t0 - 2 * HALO + r;
      float xv[KW];
#pragma unroll
      for (int k = 0; k < KW; ++k) xv[k] = xin[r + k];
      uint32_t o[CH / 2] = {};
      if (t >= 0 && t < L) {
        float v[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          float s = 0.0f;
#pragma unroll
          for (int k = 0; k < KW; ++k) s = fmaf(w1r[c][k], xv[k], s);
          v[c] = fmaxf(s + b1r[c], 0.0f);
        }
#pragma unroll
        for (int q = 0; q < CH / 2; ++q) o[q] = pack_bf16(v[2 * q], v[2 * q + 1]);
      }
      if constexpr (CH == 8) *reinterpret_cast<uint4 *>(a1 + r * I::XS + c0) = uint4{o[0], o[1], o[2], o[3]};
      else *reinterpret_cast<uint2 *>(a1 + r * I::XS + c0) = uint2{o[0], o[1]};
    }
    __syncthreads();
    if (!kShort || 32 * wave < rows + 2 * HALO) {
      conv(a1);  // layer 2: row r is time t0 - HALO + r
      const int t = t0 - HALO + row;
      const bool in = t >= 0 && t < L;
#pragma unroll
      for (int c = 0; c < I::NCO; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = in ? fmaxf(acc[c][4 * q + u] + bias(b2, c, 4 * q + u), 0.0f) : 0.0f;
          *reinterpret_cast<uint2 *>(a2 + row * I::XS + 32 * c + 8 * q + 4 * h) =
              uint2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        }
    }
    __syncthreads();  // layer 2 is complete and done with its weights
    store_w();
    load_w(0);
    __syncthreads();
    if (kShort && 32 * wave >= rows) continue;  // (this was the only tile)
    conv(a2);  // layer 3: row r is time t0 + r
    const bool in = row < rows;
#pragma unroll
    for (int c = 0; c < I::NCO; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[c][v] += in ? fmaxf(acc[c][v] + bias(b3, c, v), 0.0f) : 0.0f;
  }
  // sums over the 32 columns of a lane half, then over the waves
  float *red = reinterpret_cast<float *>(a1);  // [wave][C]
  __syncthreads();
#pragma unroll
  for (int c = 0; c < I::NCO; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      float s = sum[c][v];
#pragma unroll
      for (int m = 1; m < 32; m <<= 1) s += __shfl_xor(s, m);
      if (n == 0) red[wave * C + 32 * c + 8 * (v >> 2) + 4 * h + (v & 3)] = s;
    }
  __syncthreads();
  if (tid < C)
    part[(static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * C + tid] =
        ((red[tid] + red[C + tid]) + (red[2 * C + tid] + red[3 * C + tid])) +
        ((red[4 * C + tid] + red[5 * C + tid]) + (red[6 * C + tid] + red[7 * C + tid]));
}

// logits[b][j] = bo[j] + sum_c wo[j][c] g[c], g the mean over time from the splits' sums.
__global__ __launch_bounds__(64) void k_pool_parts(const float *__restrict__ part, int splits, int C, int L,
                                                   const float *__restrict__ wo, const float *__restrict__ bo,
                                                   float *__restrict__ logits) {
  __shared__ float gs[64];
  const int b = blockIdx.x, c = threadIdx.x;
  if (c < C) {
    float s = 0.0f;
    for (int i = 0; i < splits; ++i) s += part[(static_cast<int64_t>(b) * splits + i) * C + c];
    gs[c] = s / static_cast<float>(L);
  }
  __syncthreads();
  if (c < NCLS) {
    float v = bo[c];
    for (int i = 0; i < C; ++i) v = fmaf(wo[c * C + i], gs[i], v);
    logits[static_cast<int64_t>(b) * NCLS + c] = v;
  }
}

// Partial weight gradients of one slice of (series, time) of a C -> C layer:
// part[slice][k][co][ci] = sum of dz[b][t][co] x[b][t + k - HALO][ci] and
// part_b[slice][co] = sum of dz[b][t][co], C x C and C values (padded to the
// tiles of 32 they left room for one slice at C = 1: one wave did the whole
// batch, 3.6 ms for 8 series of 1500).
// kMask: dz is given as z > 0 ? chan[b][c] : 0.
//
// One wave per pair of channel tiles: lane (n, h) feeds channel n of both
// operands at the time steps of parity h, straight from memory (32 channels
// are one 128-byte line), and one sliding window of x serves all seven taps:
// 12 loads per 28 products of 64 cycles, so the matrix cores bound it.  (The
// VALU form took 1.2 ms per layer at C = 64, 256 x 1500, and as long for the
// first layer's 7 x 64 weights.)
constexpr int WT = 128;         // time steps of a slice's unit
constexpr int kSlices64 = 512;  // slices at C > 32 (four waves each), at most
template <int NCO, bool kMask>
__global__ __launch_bounds__(64 * NCO * NCO) void k_wgrad(const float *__restrict__ x, const float *__restrict__ dz,
                                                          const float *__restrict__ chan, int C, int L,
                                                          int64_t units, int64_t units_per_slice,
                                                          float *__restrict__ part, float *__restrict__ part_b) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int cot = wave % NCO, cit = wave / NCO;
  const int co = 32 * cot + n, ci = 32 * cit + n;
  const bool has_co = co < C, has_ci = ci < C;
  f32x16_t acc[KW];
#pragma unroll
  for (int k = 0; k < KW; ++k) acc[k] = f32x16_t{};
  float bsum = 0.0f;
  const int per_series = (L + WT - 1) / WT;
  const int64_t u0 = static_cast<int64_t>(blockIdx.x) * units_per_slice;
  const int64_t u1 = u0 + units_per_slice < units ? u0 + units_per_slice : units;
  for (int64_t u = u0; u < u1; ++u) {
    const int b = static_cast<int>(u / per_series);
    const int t0 = static_cast<int>(u - static_cast<int64_t>(b) * per_series) * WT;
    const float *xb = x + static_cast<int64_t>(b) * L * C + (has_ci ? ci : 0);
    const float *zb = dz + static_cast<int64_t>(b) * L * C + (has_co ? co : 0);
    float cz = 0.0f;
    if constexpr (kMask) cz = has_co ? chan[b * C + co] : 0.0f;
    // Loads are unconditional (clamped) and two groups ahead; what lies outside
    // the series or the channels is replaced when a group becomes current.
    auto raw_x = [&](int t) { return xb[static_cast<int64_t>(t < 0 ? 0 : (t < L ? t : L - 1)) * C]; };
    auto raw_z = [&](int t) { return zb[static_cast<int64_t>(t < L ? t : L - 1) * C]; };
    auto use_x = [&](float v, int t) { return has_ci && t >= 0 && t < L ? v : 0.0f; };
    auto use_z = [&](float v, int t) {
      if constexpr (kMask) v = v > 0.0f ? cz : 0.0f;
      return has_co && t < L ? v : 0.0f;
    };
    // groups of 4 steps (8 time steps); step i of the group at T covers time
    // T + 2 i + h and needs x at that time - 3 .. + 3
    const int th = t0 + h;
    float xw[13], zw[4], x1[8], z1[4];  // this group's, and the next one's (raw)
#pragma unroll
    for (int i = 0; i < 13; ++i) xw[i] = raw_x(th - HALO + i);
#pragma unroll
    for (int i = 0; i < 4; ++i) zw[i] = raw_z(th + 2 * i);
#pragma unroll
    for (int i = 0; i < 8; ++i) x1[i] = raw_x(th + 8 - HALO + 5 + i);
#pragma unroll
    for (int i = 0; i < 4; ++i) z1[i] = raw_z(th + 8 + 2 * i);
#pragma unroll
    for (int i = 0; i < 13; ++i) xw[i] = use_x(xw[i], th - HALO + i);
#pragma unroll
    for (int i = 0; i < 4; ++i) zw[i] = use_z(zw[i], th + 2 * i);
    const int te = L - t0 < WT ? L - t0 : WT;
#pragma unroll 1
    for (int T = 0; T < te; T += 8) {
      float x2[8], z2[4];  // two groups ahead (raw)
#pragma unroll
      for (int i = 0; i < 8; ++i) x2[i] = raw_x(th + T + 16 - HALO + 5 + i);
#pragma unroll
      for (int i = 0; i < 4; ++i) z2[i] = raw_z(th + T + 16 + 2 * i);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bsum += zw[i];
#pragma unroll
        for (int k = 0; k < KW; ++k)
          acc[k] = __builtin_amdgcn_mfma_f32_32x32x2f32(zw[i], xw[2 * i + k], acc[k], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 5; ++i) xw[i] = xw[i + 8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        xw[5 + i] = use_x(x1[i], th + T + 8 - HALO + 5 + i);
        x1[i] = x2[i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        zw[i] = use_z(z1[i], th + T + 8 + 2 * i);
        z1[i] = z2[i];
      }
    }
  }
  float *out = part + static_cast<int64_t>(blockIdx.x) * KW * C * C;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int o = 32 * cot + 8 * (v >> 2) + 4 * h + (v & 3);
    if (o >= C || !has_ci) continue;
#pragma unroll
    for (int k = 0; k < KW; ++k) out[(k * C + o) * C + ci] = acc[k][v];
  }
  bsum += __shfl_xor(bsum, 32);
  if (cit == 0 && h == 0 && has_co) part_b[static_cast<int64_t>(blockIdx.x) * C + co] = bsum;
}

// Layer 1's partial gradients: part[slice][c][k < KW] weights, [c][KW] the
// bias.  Bound by reading dz once; a thread holds one channel of one residue
// of time modulo 4.
constexpr int kSlices1 = 2048;
__global__ __launch_bounds__(256) void k_wgrad1(const float *__restrict__ x, int64_t ldx, const float *__restrict__ dz,
                                                int C, int L, int64_t units, int64_t units_per_slice,
                                                float *__restrict__ part) {
  __shared__ float xs[WT + KW - 1];
  __shared__ float red[4][kMaxC][KW + 1];
  const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
  float acc[KW + 1];
#pragma unroll
  for (int k = 0; k <= KW; ++k) acc[k] = 0.0f;
  const int per_series = (L + WT - 1) / WT;
  const int64_t u0 = static_cast<int64_t>(blockIdx.x) * units_per_slice;
  const int64_t u1 = u0 + units_per_slice < units ? u0 + units_per_slice : units;
  for (int64_t u = u0; u < u1; ++u) {
    const int b = static_cast<int>(u / per_series);
    const int t0 = static_cast<int>(u - static_cast<int64_t>(b) * per_series) * WT;
    __syncthreads();
    static_assert(WT + KW - 1 <= 256, "one thread per staged sample");
    if (threadIdx.x < WT + KW - 1) {
      const int t = t0 + static_cast<int>(threadIdx.x) - HALO;
      xs[threadIdx.x] = t >= 0 && t < L ? x[static_cast<int64_t>(b) * ldx + t] : 0.0f;
    }
    __syncthreads();
    const int te = L - t0 < WT ? L - t0 : WT;
    const float *z = dz + (static_cast<int64_t>(b) * L + t0) * C + (c < C ? c : 0);
#pragma unroll 8
    for (int t = q; t < te; t += 4) {
      const float v = z[static_cast<int64_t>(t) * C];
#pragma unroll
      for (int k = 0; k < KW; ++k) acc[k] = fmaf(v, xs[t + k], acc[k]);
      acc[KW] += v;
    }
  }
#pragma unroll
  for (int k = 0; k <= KW; ++k) red[q][c][k] = acc[k];
  __syncthreads();
  for (int i = threadIdx.x; i < C * (KW + 1); i += 256) {
    const int cc = i / (KW + 1), k = i % (KW + 1);
    part[static_cast<int64_t>(blockIdx.x) * C * (KW + 1) + i] =
        (red[0][cc][k] + red[1][cc][k]) + (red[2][cc][k] + red[3][cc][k]);
  }
}

// Sum of the slices' value i of n, by the workgroup's 4 waves (64 values each
// workgroup, slices modulo 4 per wave); valid in wave 0.
__device__ __forceinline__ float sum_slices(const float *__restrict__ part, int64_t n, int slices, int64_t i) {
  __shared__ float red[4][64];
  const int q = threadIdx.x >> 6, l = threadIdx.x & 63;
  float v = 0.0f;
  if (i < n) {
#pragma unroll 8
    for (int s = q; s < slices; s += 4) v += part[static_cast<int64_t>(s) * n + i];
  }
  red[q][l] = v;
  __syncthreads();
  v = (red[0][l] + red[1][l]) + (red[2][l] + red[3][l]);
  __syncthreads();
  return v;
}

// dw[co][ci][k] and db[co] of a C -> C layer from k_wgrad's slices.
__global__ __launch_bounds__(256) void k_sum_wgrad(const float *__restrict__ part, const float *__restrict__ part_b,
                                                   int C, int slices, float *__restrict__ dw,
                                                   float *__restrict__ db) {
  const int n = KW * C * C;
  const int i = static_cast<int>(blockIdx.x) * 64 + static_cast<int>(threadIdx.x & 63);
  const bool tail = blockIdx.x + 1 == gridDim.x;  // the last workgroup sums the bias
  const int c = static_cast<int>(threadIdx.x & 63);
  const float v = tail ? sum_slices(part_b, C, slices, c) : sum_slices(part, n, slices, i);
  if (threadIdx.x >= 64) return;
  if (tail) {
    if (c < C) db[c] = v;
  } else if (i < n) {
    const int ci = i % C, co = i / C % C, k = i / (C * C);
    dw[(co * C + ci) * KW + k] = v;
  }
}

__global__ __launch_bounds__(256) void k_sum_wgrad1(const float *__restrict__ part, int C, int slices,
                                                    float *__restrict__ dw, float *__restrict__ db) {
  const int64_t n = static_cast<int64_t>(C) * (KW + 1);
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 64 + (threadIdx.x & 63);
  const float v = sum_slices(part, n, slices, i);
  if (threadIdx.x >= 64 || i >= n) return;
  const int c = static_cast<int>(i / (KW + 1)), k = static_cast<int>(i % (KW + 1));
  if (k < KW) dw[c * KW + k] = v;
  else db[c] = v;
}

// g[b][c] = mean_t a[b][t][c]; logits[b][j] = bo[j] + sum_c wo[j][c] g[b][c].
// One workgroup per series, its threads dealt out over channels and time steps.
__global__ __launch_bounds__(1024) void k_pool_linear(const float *__restrict__ a, int C, int L,
                                                      const float *__restrict__ wo, const float *__restrict__ bo,
                                                      float *__restrict__ g, float *__restrict__ logits) {
  __shared__ float red[1024];
  __shared__ float gs[kMaxC];
  const int b = blockIdx.x, tid = threadIdx.x;
  const int lgc = lg_lanes(C), c = tid & ((1 << lgc) - 1), rows = 1024 >> lgc;
  float s = 0.0f;
  if (c < C) {
    const float *row = a + static_cast<int64_t>(b) * L * C + c;
#pragma unroll 8
    for (int t = tid >> lgc; t < L; t += rows) s += row[static_cast<int64_t>(t) * C];
  }
  red[tid] = s;
  __syncthreads();
  if (tid < C) {
    float v = 0.0f;
#pragma unroll 16
    for (int i = 0; i < rows; ++i) v += red[(i << lgc) + tid];
    gs[tid] = v / static_cast<float>(L);
    g[static_cast<int64_t>(b) * C + tid] = gs[tid];
  }
  __syncthreads();
  if (tid < NCLS) {
    float v = bo[tid];
    for (int i = 0; i < C; ++i) v = fmaf(wo[tid * C + i], gs[i], v);
    logits[static_cast<int64_t>(b) * NCLS + tid] = v;
  }
}

// Softmax cross-entropy per series: loss_b[b], dlog[b][j] = (p_j - [j == y]) / B.
__global__ void k_softmax_ce(const float *__restrict__ logits, const int32_t *__restrict__ labels,
                             int B, float *__restrict__ loss_b, float *__restrict__ dlog) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const float *z = logits + static_cast<int64_t>(b) * NCLS;
  float mx = z[0];
  for (int j = 1; j < NCLS; ++j) mx = fmaxf(mx, z[j]);
  float s = 0.0f;
  for (int j = 0; j < NCLS; ++j) s += expf(z[j] - mx);
  int y = labels[b] - 1;
  y = y < 0 ? 0 : (y >= NCLS ? NCLS - 1 : y);  // labels are validated on the host
  loss_b[b] = logf(s) - (z[y] - mx);
  for (int j = 0; j < NCLS; ++j)
    dlog[static_cast<int64_t>(b) * NCLS + j] = (expf(z[j] - mx) / s - (j == y ? 1.0f : 0.0f)) / B;
}

// Output-layer gradients, one wave per weight: dwo[j][c], then dbo[j].
__global__ __launch_bounds__(256) void k_linear_bwd(const float *__restrict__ dlog, const float *__restrict__ g, int B,
                                                    int C, float *__restrict__ dwo, float *__restrict__ dbo) {
  const int e = static_cast<int>(blockIdx.x) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (e >= NCLS * (C + 1)) return;
  const int j = e / (C + 1), c = e - j * (C + 1);
  float v = 0.0f;
  for (int b = lane; b < B; b += 64)
    v = fmaf(dlog[b * NCLS + j], c < C ? g[static_cast<int64_t>(b) * C + c] : 1.0f, v);
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
  if (lane != 0) return;
  if (c < C) dwo[j * C + c] = v;
  else dbo[j] = v;
}

// Pool backward: the gradient of every time step of channel c, where its
// activation is positive: dch[b][c] = sum_j dlog[b][j] wo[j][c] / L.
__global__ void k_pool_bwd(const float *__restrict__ dlog, const float *__restrict__ wo, int64_t B, int C, int L,
                           float *__restrict__ dch) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= B * C) return;
  const int b = static_cast<int>(e / C), c = static_cast<int>(e - static_cast<int64_t>(b) * C);
  float dg = 0.0f;
#pragma unroll
  for (int j = 0; j < NCLS; ++j) dg = fmaf(dlog[b * NCLS + j], wo[j * C + c], dg);
  dch[e] = dg / static_cast<float>(L);
}

__global__ void k_mean(const float *__restrict__ v, int n, float *__restrict__ out) {
  __shared__ float s[256];
  float a = 0.0f;
  for (int i = threadIdx.x; i < n; i += 256) a += v[i];
  s[threadIdx.x] = a;
  __syncthreads();
  for (int m = 128; m > 0; m >>= 1) {
    if (static_cast<int>(threadIdx.x) < m) s[threadIdx.x] += s[threadIdx.x + m];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = s[0] / static_cast<float>(n);
}

// Adam (Kingma & Ba) with bias correction.
__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                       float c1, float c2) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

unsigned blocks_for(int64_t n, int t) {
  int64_t b = (n + t - 1) / t;
  if (b < 1) b = 1;
  if (b > 65536) b = 65536;
  return static_cast<unsigned>(b);
}

}  // namespace

int64_t net_param_count(int C) { return static_cast<int64_t>(KW) * C + C + 2 * (static_cast<int64_t>(C) * C * KW + C) + NCLS * C + NCLS; }

NetParams net_params(const float *theta, int C) {
  NetParams p;
  const float *q = theta;
  p.w1 = q; q += static_cast<int64_t>(C) * KW;
  p.b1 = q; q += C;
  p.w2 = q; q += static_cast<int64_t>(C) * C * KW;
  p.b2 = q; q += C;
  p.w3 = q; q += static_cast<int64_t>(C) * C * KW;
  p.b3 = q; q += C;
  p.wo = q; q += static_cast<int64_t>(NCLS) * C;
  p.bo = q;
  return p;
}

namespace {
// Workspace of a training pass (floats).
struct NetWs {
  int64_t act, slices, slices1, units;
  int64_t a1, a2, a3, d2, g, dch, logits, dlog, loss_b, wf, part, part_b, part1, total;
  NetWs(int C, int64_t B, int64_t L, int64_t limit) {
    act = B * C * L;
    const int64_t weights = static_cast<int64_t>(KW) * C * C;
    units = B * ((L + WT - 1) / WT);
    // the partial gradients take the room that a stored gradient of the pooled
    // layer would: more slices than that do not pay for their sums
    const int64_t most = C > 32 ? kSlices64 : 4 * kSlices64;
    const int64_t room = (act + kNetSlices * static_cast<int64_t>(C) * (C * KW + 1)) / (weights + C);
    slices = units < most ? units : most;
    slices = slices < room ? slices : room;
    slices = slices > 1 ? slices : 1;
    slices1 = units < kSlices1 ? units : kSlices1;
    lay_out(C, B);
    if (total <= limit) return;
    // the room beside one slice each: a quarter for layer 1, the rest for the other layers
    const int64_t all = slices, all1 = slices1;
    slices = slices1 = 1;
    lay_out(C, B);
    const int64_t spare = limit > total ? limit - total : 0;  // (sizes are rounded up to 64)
    slices1 = 1 + spare / 4 / (C * (KW + 1) + 64);
    slices1 = slices1 < all1 ? slices1 : all1;
    slices = 1 + (spare - (slices1 - 1) * (C * (KW + 1) + 64)) / (weights + C + 128);
    slices = slices < all ? slices : all;
    lay_out(C, B);
  }
  void lay_out(int C, int64_t B) {
    const int64_t weights = static_cast<int64_t>(KW) * C * C;
    int64_t at = 0;
    auto take = [&](int64_t n) {
      const int64_t o = at;
      at += (n + 63) / 64 * 64;
      return o;
    };
    a1 = take(act); a2 = take(act); a3 = take(act); d2 = take(act);
    g = take(B * C); dch = take(B * C);
    logits = take(B * NCLS); dlog = take(B * NCLS); loss_b = take(B);
    wf = take(4 * frag_floats(C));
    part = take(slices * weights); part_b = take(slices * C); part1 = take(slices1 * C * (KW + 1));
    total = at;
  }
};

template <bool kBack, bool kMask>
hipError_t launch_conv(const float *x, const float *chan, int C, int64_t B, int64_t L, const float *wf,
                       const float *bias, const float *aprev, float *y, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>((L + CR - 1) / CR), static_cast<unsigned>(B));
  const f32x4_t *w = reinterpret_cast<const f32x4_t *>(wf);
  const size_t shm = sizeof(float) * (CR + KW - 1) * (pad32(C) + 1);
  if (C > 32) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_conv_f32<2, kBack, kMask>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(shm));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_conv_f32<2, kBack, kMask>), grid, dim3(256), shm, st, x, chan, C, static_cast<int>(L), w,
                       bias, aprev, y);
  } else {
    hipLaunchKernelGGL((k_conv_f32<1, kBack, kMask>), grid, dim3(256), shm, st, x, chan, C, static_cast<int>(L), w,
                       bias, aprev, y);
  }
  return hipGetLastError();
}

template <bool kMask>
hipError_t launch_wgrad(const NetWs &W, const float *x, const float *dz, const float *chan, int C, int64_t L,
                        float *ws, float *dw, float *db, hipStream_t st) {
  const int64_t per = (W.units + W.slices - 1) / W.slices;
  const unsigned used = static_cast<unsigned>((W.units + per - 1) / per);  // slices with work
  if (C > 32)
    hipLaunchKernelGGL((k_wgrad<2, kMask>), dim3(used), dim3(256), 0, st, x, dz, chan, C, static_cast<int>(L), W.units,
                       per, ws + W.part, ws + W.part_b);
  else
    hipLaunchKernelGGL((k_wgrad<1, kMask>), dim3(used), dim3(64), 0, st, x, dz, chan, C, static_cast<int>(L), W.units,
                       per, ws + W.part, ws + W.part_b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  static_assert(kMaxC <= 64, "one workgroup sums the bias");
  const unsigned gx = static_cast<unsigned>((KW * C * C + 63) / 64 + 1);
  hipLaunchKernelGGL(k_sum_wgrad, dim3(gx), dim3(256), 0, st, ws + W.part, ws + W.part_b, C, static_cast<int>(used),
                     dw, db);
  return hipGetLastError();
}

// Forward pass (net_forward), with the flipped weights too for a training pass.
hipError_t forward(const float *theta, int C, const float *X, int64_t B, int64_t L, int64_t ldx, float *ws,
                   int64_t limit, float *logits, bool train, hipStream_t st) {
  const NetParams P = net_params(theta, C);
  const NetWs W(C, B, L, limit);
  const int frags = frag_floats(C);
  static_assert(frag_floats(1) % 256 == 0 && frag_floats(kMaxC) % 256 == 0, "whole workgroups of weights");
  float *a1 = ws + W.a1, *a2 = ws + W.a2, *a3 = ws + W.a3, *wf = ws + W.wf;
  const int64_t wgs = B * ((L + T1 - 1) / T1) + (train ? 4 : 2) * (frags / 256);
  if (wgs > 0x7fffffff) return hipErrorInvalidValue;  // (far above what the workspace limit lets in)
  hipLaunchKernelGGL(k_conv1, dim3(static_cast<unsigned>(wgs)), dim3(256), 0, st, X, ldx, static_cast<int>(B), C,
                     static_cast<int>(L), P.w1, P.b1, a1, P.w2, P.w3, wf);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = launch_conv<false, false>(a1, nullptr, C, B, L, wf, P.b2, nullptr, a2, st);
  if (e == hipSuccess) e = launch_conv<false, false>(a2, nullptr, C, B, L, wf + frags, P.b3, nullptr, a3, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_pool_linear, dim3(static_cast<unsigned>(B)), dim3(1024), 0, st, a3, C, static_cast<int>(L), P.wo,
                     P.bo, ws + W.g, logits);
  return hipGetLastError();
}
}  // namespace

int64_t net_limit_floats(int C, int64_t B, int64_t L) {
  return 5 * B * C * L + B * C + 3 * B * NCLS + B + kNetSlices * (static_cast<int64_t>(C) * C * KW + C) + 64;
}

int64_t net_workspace_floats(int C, int64_t B, int64_t L, int64_t limit) { return NetWs(C, B, L, limit).total; }

hipError_t net_forward(const float *theta, int C, const float *X, int64_t B, int64_t L,
                       int64_t ldx, float *ws, int64_t limit, float *logits, hipStream_t st) {
  return forward(theta, C, X, B, L, ldx, ws, limit, logits, false, st);
}

namespace {
// Tiles of a series and the workgroups that share them.
int infer_tiles(int64_t L) { return static_cast<int>((L + TO - 1) / TO); }
int infer_splits(int64_t B, int64_t L) {
  const int64_t want = (kInferWgs + B - 1) / B;
  return static_cast<int>(want < infer_tiles(L) ? want : infer_tiles(L));
}

int64_t infer_words(int C) { return C == 64 ? Infer<64>::NW : Infer<32>::NW; }

template <int C>
hipError_t launch_infer(const NetParams &P, const float *X, int64_t B, int64_t L, int64_t ldx, const uint16_t *wb,
                        float *part, hipStream_t st) {
  constexpr size_t shm = Infer<C>::lds;
  const auto fn = L <= TO - 32 ? &k_net_infer<C, true> : &k_net_infer<C, false>;
  if (shm > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(shm));
    if (e != hipSuccess) return e;
  }
  const dim3 grid(static_cast<unsigned>(infer_splits(B, L)), static_cast<unsigned>(B));
  hipLaunchKernelGGL(fn, grid, dim3(IT), shm, st, X, ldx, static_cast<int>(L), P.w1, P.b1, P.b2, P.b3,
                     reinterpret_cast<const u32x4_t *>(wb), infer_tiles(L), part);
  return hipGetLastError();
}
}  // namespace

int64_t net_infer_workspace_floats(int C, int64_t B, int64_t L) {
  // BF16 weights of two layers, sums per split
  return 2 * 4 * infer_words(C) + B * infer_splits(B, L) * C;
}

hipError_t net_forward_bf16(const float *theta, int C, const float *X, int64_t B, int64_t L,
                            int64_t ldx, float *ws, float *logits, hipStream_t st) {
  if (C != 32 && C != 64) return hipErrorInvalidValue;
  const NetParams P = net_params(theta, C);
  uint16_t *wb = reinterpret_cast<uint16_t *>(ws);  // the workspace is 256-byte aligned
  const int words = static_cast<int>(infer_words(C));
  float *part = ws + 2 * 4 * words;
  hipLaunchKernelGGL(k_w_to_bf16, dim3(static_cast<unsigned>(2 * words * 8 / 256)), dim3(256), 0, st, P.w2, P.w3, C,
                     words, wb);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = C == 64 ? launch_infer<64>(P, X, B, L, ldx, wb, part, st) : launch_infer<32>(P, X, B, L, ldx, wb, part, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_pool_parts, dim3(static_cast<unsigned>(B)), dim3(64), 0, st, part, infer_splits(B, L), C,
                     static_cast<int>(L), P.wo, P.bo, logits);
  return hipGetLastError();
}

hipError_t net_loss_grad(const float *theta, int C, const float *X, const int32_t *labels,
                         int64_t B, int64_t L, int64_t ldx, float *ws, int64_t limit, float *loss,
                         float *grad, hipStream_t st) {
  const NetParams P = net_params(theta, C), G = net_params(grad, C);
  const NetWs W(C, B, L, limit);
  auto mut = [](const float *p) { return const_cast<float *>(p); };
  float *a1 = ws + W.a1, *a2 = ws + W.a2, *a3 = ws + W.a3, *d2 = ws + W.d2;
  float *g = ws + W.g, *dch = ws + W.dch, *logits = ws + W.logits, *dlog = ws + W.dlog, *loss_b = ws + W.loss_b;
  const float *wf3 = ws + W.wf + 2 * frag_floats(C), *wf2 = ws + W.wf + 3 * frag_floats(C);
  hipError_t e = forward(theta, C, X, B, L, ldx, ws, limit, logits, true, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_softmax_ce, dim3(blocks_for(B, 128)), dim3(128), 0, st, logits, labels, static_cast<int>(B), loss_b, dlog);
  hipLaunchKernelGGL(k_mean, dim3(1), dim3(256), 0, st, loss_b, static_cast<int>(B), loss);
  hipLaunchKernelGGL(k_linear_bwd, dim3(static_cast<unsigned>((NCLS * (C + 1) + 3) / 4)), dim3(256), 0, st, dlog, g,
                     static_cast<int>(B), C, mut(G.wo), mut(G.bo));
  hipLaunchKernelGGL(k_pool_bwd, dim3(static_cast<unsigned>((B * C + 255) / 256)), dim3(256), 0, st, dlog, P.wo, B, C,
                     static_cast<int>(L), dch);
  e = hipGetLastError();
  // layer 3: its gradient is dch where a3 > 0
  if (e == hipSuccess) e = launch_wgrad<true>(W, a2, a3, dch, C, L, ws, mut(G.w3), mut(G.b3), st);
  if (e == hipSuccess) e = launch_conv<true, true>(a3, dch, C, B, L, wf3, nullptr, a2, d2, st);
  // layer 2, then layer 1 (its gradient takes the place of a3)
  if (e == hipSuccess) e = launch_wgrad<false>(W, a1, d2, nullptr, C, L, ws, mut(G.w2), mut(G.b2), st);
  float *d1 = a3;
  if (e == hipSuccess) e = launch_conv<true, false>(d2, nullptr, C, B, L, wf2, nullptr, a1, d1, st);
  if (e != hipSuccess) return e;
  const int64_t per = (W.units + W.slices1 - 1) / W.slices1;
  const unsigned used = static_cast<unsigned>((W.units + per - 1) / per);
  hipLaunchKernelGGL(k_wgrad1, dim3(used), dim3(256), 0, st, X, ldx, d1, C, static_cast<int>(L), W.units, per,
                     ws + W.part1);
  hipLaunchKernelGGL(k_sum_wgrad1, dim3(static_cast<unsigned>((C * (KW + 1) + 63) / 64)), dim3(256), 0, st,
                     ws + W.part1, C, static_cast<int>(used), mut(G.w1), mut(G.b1));
  return hipGetLastError();
}

hipError_t net_adam(float *p, const float *g, float *m, float *v, int64_t n, int step, float lr,
                    float b1, float b2, float eps, hipStream_t st) {
  const float c1 = 1.0f - powf(b1, static_cast<float>(step));
  const float c2 = 1.0f - powf(b2, static_cast<float>(step));
  hipLaunchKernelGGL(k_adam, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, p, g, m, v, n, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace edm
