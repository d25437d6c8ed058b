// Host-side handle shared by the translation units of libhashgrid.
#pragma once

#include "hashgrid.h"
#include "hashgrid_common.hpp"

namespace hg {

// Plan of the binned backward pass (see bwd_binned.hip): how each level's
// gradient slice is cut into chunks that fit the LDS of one workgroup.
struct BinPlan {
  uint32_t bin_base[HG_MAX_LEVELS + 1];  // first global bin of the level; [L] = number of bins
  uint32_t wg_base[HG_MAX_LEVELS + 1];   // first accumulate-workgroup of the level; [L] = their number
  uint32_t slices[HG_MAX_LEVELS];        // workgroups that share one bin of the level
  uint32_t group_mask;                   // levels whose work items are shared out by features as well (accumulate pass)
  // 1:1 levels: log2 of grid rows per chunk (32 bits: the scalar unit loads no bytes, and to wait for a vector load
  // is to wait for every gather before it: encode at 2^18 points, d = 2, T = 2^22: 287.2 -> 282.5 us with 8 -> 32 bits)
  uint32_t row_shift[HG_MAX_LEVELS];
  uint32_t chunk_log2;                   // log2 of the entries a chunk can hold
  uint32_t rec_per_point;                // records per (point, level) at most: 2^(d-1) pairs of corners, or 2^d corners
  uint32_t corner_records;               // 1: every level cut into aligned blocks of 2^chunk_log2 entries, a pair's corners have
                                         // a record each where one cannot name both (T not a power of two, or d = 1); 0: one per pair
  uint32_t count_parts, scatter_parts;   // level parts (gridDim.y) of the count and scatter grids
  uint32_t tile_mult;                    // a tile of the sort = tile_mult * 512 points (of a batch: tile_mult_for); above 2: no
                                         // staging (bin_scatter_direct)
  uint32_t supported;                    // 0: configuration not served by the binned path
};

}  // namespace hg

struct hashgrid {
  hashgrid_config cfg;
  hg::LevelTable lv;
  uint64_t total;
  hg::BinPlan bp;
};

namespace hg {
void build_bin_plan(hashgrid* h);
// bwd_binned.hip: the plan's tile_mult for a batch of B points: 2 where 1 would leave few records to a bin
uint32_t tile_mult_for(const hashgrid* h, uint32_t B);
// hashgrid.hip: compute units of the current device at the first call
uint32_t cu_count();
// hashgrid.hip: threads (= points) per workgroup of the point-major kernels for a batch of B points
uint32_t point_major_block(uint32_t B);
// hashgrid.hip: parts of the levels that the plain forward's workgroups of a batch of B points are split over
uint32_t level_parts(uint32_t d, uint32_t T, uint32_t entry_bytes, uint32_t B);
// hashgrid.hip: forward pass that also fills counts[n_tiles][n_bins] of the binned backward pass
hg_status launch_fwd_counting(const hashgrid* h, uint32_t B, const float* x, const void* params, void* y,
                              uint32_t* counts, uint32_t n_bins, uint32_t n_tiles, hipStream_t s);

struct AdamArgs;
struct AdamState;
struct SideJob;
// mlp_bwd.hip: the network's part of a training step, forward products, loss and backward products (shapes as
// hashgrid_mlp_bwd takes them, checked by the caller).  Every workgroup (kMaxMlpGroups at most) leaves its loss
// and weight-gradient sums in scratch (HG_TRAIN_SCRATCH_BYTES); fills in where they are in *job.
constexpr uint32_t kMaxMlpGroups = 256;
hg_status launch_mlp_train(uint32_t B, uint32_t n_in, uint32_t n_out, const void* y, const void* W1, const void* W2,
                           const void* W3, const float* target, uint32_t loss, float scale, void* dLdy, SideJob* job,
                           void* scratch, hipStream_t s);

// bwd_binned.hip: the sorted backward pass that hands every entry's sum to the optimiser instead of to a gradient array
// (io fp16, gradients fp32, pair records; workspace checked by the caller).  zeros: n_entries * F floats that are all
// zero, and are again after the call: where several workgroups share a chunk their sums meet there.
hg_status launch_binned_adam(const hashgrid* h, uint32_t B, const float* x, const void* dy, float* zeros, void* workspace,
                             bool counted, const AdamArgs& a, const AdamState& st, const SideJob& job, hipStream_t s);
// hashgrid.hip: the optimiser's step on the entries that the batch's corners reach (d = 2 or 3); grad is all zeros after it
hg_status launch_adam_touched(const hashgrid* h, uint32_t B, const float* x, float* grad, const AdamArgs& a,
                              const AdamState& st, const SideJob& job, hipStream_t s);
}
