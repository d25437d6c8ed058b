// One scalar's training loss (paper Section 4, "Training"), shared by the loss kernel (loss.hip) and the network's
// training kernel, which takes it between its forward and backward products (mlp_bwd.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "hashgrid.h"

namespace hg {

constexpr float kMapeOffset = 0.01f;  // Section 4, "Training": the constant in the percentage error's denominator

// value and slope of one scalar's loss; fp32, the sign of p - t is exact (a difference of two floats
// is zero only if they are equal)
template <int KIND>
__device__ __forceinline__ void loss_scalar(float p, float t, float scale, float& slope, float& value) {
  const float diff = p - t;
  if (KIND == HG_LOSS_L2) {
    value = diff * diff;
    slope = scale * (2.0f * diff);
  } else {
    const float inv = 1.0f / (fabsf(t) + kMapeOffset);
    value = fabsf(diff) * inv;
    slope = diff > 0.0f ? scale * inv : (diff < 0.0f ? -(scale * inv) : diff);  // diff itself where it is 0 or NaN
  }
}

}  // namespace hg
