// The optimiser step on one scalar (paper Section 4, "Training"), shared by the kernels that apply it: the streaming
// one over whole arrays (adam.hip), the accumulate pass that owns a chunk of the gradient (bwd_binned.hip) and the
// one that visits only what a small batch touched (train.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hashgrid.h"

namespace hg {

struct AdamArgs {
  float lr, beta1, beta2, eps, l2;
  float inv_c1;       // 1 / (1 - beta1^t)
  float inv_sqrt_c2;  // 1 / sqrt(1 - beta2^t)
};

// adam.hip: the checks every entry point makes of the hyper-parameters, and the step's factors
bool adam_config_ok(const hashgrid_adam_config& cfg);
AdamArgs adam_args(const hashgrid_adam_config& cfg, uint32_t step);

__device__ __forceinline__ void adam_scalar(const AdamArgs& a, float g, float& m, float& v, float& p) {
  m = a.beta1 * m + (1.0f - a.beta1) * g;
  v = a.beta2 * v + (1.0f - a.beta2) * g * g;
  p -= a.lr * (m * a.inv_c1) / (sqrtf(v) * a.inv_sqrt_c2 + a.eps);
}

// What the optimiser keeps beside a gradient: the full-precision master copy, the half-precision working copy
// (may be null) and both moments.
struct AdamState {
  float* p32;
  _Float16* p16;
  float* m;
  float* v;
};

// Work that a training step's later kernel does on the side, in workgroups of its own: Adam on the network's weights (a
// few thousand scalars, each gradient cleared as it is read) and the sum of the loss values that the workgroups of the network kernel left.
// A launch of its own for either costs more than the work.  blocks = 0: nothing to do.
struct SideJob {
  uint32_t blocks;  // workgroups appended to the grid
  uint32_t n;
  AdamArgs a;
  AdamState w;
  float* grad;
  const double* loss_parts;
  uint32_t n_parts;
  double* loss_sum;
};

// One workgroup's share (block = 0 .. job.blocks - 1); every thread of the workgroup calls it.
__device__ __forceinline__ void run_side_job(const SideJob& job, const uint32_t block) {
  for (uint32_t i = block * blockDim.x + threadIdx.x; i < job.n; i += job.blocks * blockDim.x) {
    float p = job.w.p32[i], g = job.grad[i];
    job.grad[i] = 0.0f;
    g = job.a.l2 != 0.0f ? fmaf(job.a.l2, p, g) : g;
    if (g == 0.0f) continue;
    float m = job.w.m[i], v = job.w.v[i];
    adam_scalar(job.a, g, m, v, p);
    job.w.m[i] = m;
    job.w.v[i] = v;
    job.w.p32[i] = p;
    job.w.p16[i] = (_Float16)p;
  }
  if (block == 0 && threadIdx.x < 64) {  // one wave
    double sum = 0.0;
    for (uint32_t i = threadIdx.x; i < job.n_parts; i += 64) sum += job.loss_parts[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o, 64);
    if (threadIdx.x == 0) *job.loss_sum = sum;
  }
}

}  // namespace hg
