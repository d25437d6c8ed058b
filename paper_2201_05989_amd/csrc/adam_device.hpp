// The optimiser step on one scalar (paper Section 4, "Training"), shared by the kernels that apply it: the streaming
// one over whole arrays (adam.hip), the accumulate pass that owns a chunk of the gradient (bwd_binned.hip) and the
// one that visits only what a small batch touched (adam_touched, hashgrid.hip).
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

// How the network's weight-gradient sums lie in a workgroup of mlp_bwd.hip: `quads` runs of four registers of 64 lanes.
// Quads 0 .. 15 are the four 32 x 32 tiles of dW2 (tile 2 Tm + Tn), then 8 KB quads of dW1 (tile KB Tn + Tk: rows n of
// tile Tn, columns k of tile Tk), then 2 OS of dW3 (tile Tn: the OS runs of eight rows o that exist); register t of quad q of a
// tile holds row 8 q + 4 (lane / 32) + t at column lane % 32.
struct SumLayout {
  int kb, os, n_in, n_out;
  __host__ __device__ int quads() const { return 16 + 8 * kb + 2 * os; }
  // index into W1 [64][n_in], W2 [64][64], W3 [n_out][64] laid one after the other; -1 for padding (k >= n_in, o >= n_out)
  __device__ int scalar_of(const int i, const int t, const int lane) const {
    const int c = lane & 31, half_row = 4 * (lane >> 5) + t;
    if (i < 16) {
      const int a = i / 4, row = 8 * (i % 4) + half_row;
      return 64 * n_in + (32 * (a / 2) + row) * 64 + 32 * (a % 2) + c;
    }
    if (i < 16 + 8 * kb) {
      const int a = (i - 16) / 4, row = 8 * ((i - 16) % 4) + half_row, k = 32 * (a % kb) + c;
      return k < n_in ? (32 * (a / kb) + row) * n_in + k : -1;
    }
    const int j = i - 16 - 8 * kb, row = 8 * (j % os) + half_row;
    return row < n_out ? 64 * n_in + 64 * 64 + row * 64 + 32 * (j / os) + c : -1;
  }
};

// Work that a training step's later kernel does on the side, in workgroups of its own: the weight-gradient sums that the
// workgroups of the network kernel left are added up and taken to Adam on the network's weights, and their loss
// values are added up.  A launch of its own costs more than the work, and letting the workgroups of
// the network kernel meet in one array with atomic additions costs them 5 us at its end (every workgroup has all
// scalars, 100 K requests of 64 bytes).  blocks = 0: nothing to do; else one workgroup for every quad of sums.
struct SideJob {
  uint32_t blocks;
  SumLayout at;
  AdamArgs a;
  AdamState w;         // the weights, in the order of SumLayout::scalar_of
  const float4* sums;  // [n_parts][quads][64]
  const double* loss_parts;
  uint32_t n_parts;
  double* loss_sum;
};

// Quad `quad` of the job, by all T threads of a workgroup; `part`: T float4 of LDS.
template <int T>
__device__ __forceinline__ void run_side_job(const SideJob& job, const uint32_t quad, float4* part) {
  constexpr uint32_t kSegments = T / 64;
  const uint32_t lane = threadIdx.x & 63, seg = threadIdx.x >> 6;
  float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 8
  for (uint32_t p = seg; p < job.n_parts; p += kSegments) {
    const float4 v = job.sums[((uint64_t)p * job.blocks + quad) * 64 + lane];
    sum.x += v.x;
    sum.y += v.y;
    sum.z += v.z;
    sum.w += v.w;
  }
  part[threadIdx.x] = sum;
  __syncthreads();
  if (threadIdx.x < 256) {  // lane and register: 64 x 4 scalars
    const uint32_t t = threadIdx.x >> 6;
    float g = 0.0f;
#pragma unroll
    for (uint32_t s = 0; s < kSegments; ++s) g += reinterpret_cast<const float*>(part + s * 64 + lane)[t];
    const int i = job.at.scalar_of((int)quad, (int)t, (int)lane);
    if (i >= 0) {
      float p = job.w.p32[i];
      g = job.a.l2 != 0.0f ? fmaf(job.a.l2, p, g) : g;
      if (g != 0.0f) {
        float m = job.w.m[i], v = job.w.v[i];
        adam_scalar(job.a, g, m, v, p);
        job.w.m[i] = m;
        job.w.v[i] = v;
        job.w.p32[i] = p;
        job.w.p16[i] = (_Float16)p;
      }
    }
  }
  if (quad == 0 && threadIdx.x < 64) {  // one wave
    double total = 0.0;
    for (uint32_t i = lane; i < job.n_parts; i += 64) total += job.loss_parts[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) total += __shfl_down(total, o, 64);
    if (lane == 0) *job.loss_sum = total;
  }
}

}  // namespace hg
