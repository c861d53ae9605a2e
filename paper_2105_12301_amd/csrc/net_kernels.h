// Internal interface of the surrogate-network kernels (net.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace edm {

// Flat parameter layout: w1[C][1][KW], b1[C], w2[C][C][KW], b2[C],
// w3[C][C][KW], b3[C], wo[20][C], bo[20].
struct NetParams {
  const float *w1, *b1, *w2, *b2, *w3, *b3, *wo, *bo;
};

constexpr int kNetSlices = 64;  // (series, time) slices of a weight gradient that net_limit_floats counts with

int64_t net_param_count(int C);
NetParams net_params(const float *theta, int C);
// A call is refused where net_limit_floats, a bound of one pass over B series of
// length L with a stored gradient of the pooled layer, passes the workspace
// limit.  net_workspace_floats is what a forward/backward pass under that limit
// (floats) reserves: its slices of partial gradients are as many as the limit
// has room for.  (Up to four channels the weights' layout may pass a limit of
// less than 30 KB; a workspace is a whole number of MiB.)
int64_t net_limit_floats(int C, int64_t B, int64_t L);
int64_t net_workspace_floats(int C, int64_t B, int64_t L, int64_t limit);
// Workspace of net_forward_bf16.
int64_t net_infer_workspace_floats(int C, int64_t B, int64_t L);

// (limit: as given to net_workspace_floats)
hipError_t net_forward(const float *theta, int C, const float *X, int64_t B, int64_t L,
                       int64_t ldx, float *ws, int64_t limit, float *logits, hipStream_t st);
// Inference with the C -> C convolutions on BF16 matrix cores (C = 32 or 64);
// ws: net_infer_workspace_floats, 256-byte aligned.
hipError_t net_forward_bf16(const float *theta, int C, const float *X, int64_t B, int64_t L,
                            int64_t ldx, float *ws, float *logits, hipStream_t st);
hipError_t net_loss_grad(const float *theta, int C, const float *X, const int32_t *labels,
                         int64_t B, int64_t L, int64_t ldx, float *ws, int64_t limit, float *loss,
                         float *grad, hipStream_t st);
hipError_t net_adam(float *p, const float *g, float *m, float *v, int64_t n, int step, float lr,
                    float b1, float b2, float eps, hipStream_t st);

}  // namespace edm
