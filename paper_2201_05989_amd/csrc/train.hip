// One training iteration of the whole model (paper Section 4, "Training") behind one call: which kernels a batch
// takes, and nothing else.
//
//   large batches   forward, counting for the sort (where the batch does not give every compute unit a full workgroup the plain
//                   forward and the count pass); network forward + loss + network backward; scan (the network's
//                   Adam step and the loss sum ride along); scatter; accumulate + Adam on the tables
//   small batches   forward; network; atomic additions into an array of zeros; Adam on what they touched
//
// Five or six, and four launches of dependent kernels, each 2.6 us after the one before at the earliest and 3 us of the
// caller's time: one call per pass of the method took eleven and ten, and read and wrote the gradient of every table entry.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "hashgrid.h"
#include "hashgrid_internal.hpp"
#include "adam_device.hpp"

extern "C" hg_status hashgrid_train_step(const hashgrid_t* hg, const hashgrid_train_state* st, uint32_t B, const float* x,
                                         const float* target, void* y, void* dLdy, void* workspace,
                                         uint64_t workspace_bytes, uint32_t step, void* stream) {
  if (!hg || !st || step == 0) return HG_ERR_INVALID_ARG;
  if (B == 0) return HG_OK;
  if (B > HG_MAX_BATCH) return HG_ERR_UNSUPPORTED;
  const hashgrid_config& c = hg->cfg;
  const uint32_t n_in = c.L * c.F, n_out = st->n_out;
  if (!x || !target || !y || !dLdy || n_out == 0) return HG_ERR_INVALID_ARG;
  if (c.param_dtype != HG_F16 || c.io_dtype != HG_F16 || c.grad_dtype != HG_F32 || !hg->lv.T_is_pow2 || c.d < 2 ||
      n_in % 8 != 0 || n_in > 64 || n_out > 32)
    return HG_ERR_UNSUPPORTED;
  if (st->loss != HG_LOSS_L2 && st->loss != HG_LOSS_MAPE) return HG_ERR_INVALID_ARG;
  if (!(fabsf(st->loss_scale) < INFINITY)) return HG_ERR_INVALID_ARG;
  if (!hg::adam_config_ok(st->tables_adam) || !hg::adam_config_ok(st->weights_adam) || st->tables_adam.l2_reg != 0.0f)
    return HG_ERR_INVALID_ARG;
  auto bad = [](const void* p, uintptr_t a) { return p == nullptr || (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; };
  if (bad(x, 4) || bad(target, 4) || bad(y, 16) || bad(dLdy, 16) || bad(st->tables, 16) || bad(st->tables_half, c.F * 2 > 8 ? c.F * 2 : 8) ||
      bad(st->tables_m, 16) || bad(st->tables_v, 16) || bad(st->tables_zeros, 16) || bad(st->weights, 4) ||
      bad(st->weights_half, 8) || bad(st->weights_m, 4) || bad(st->weights_v, 4) || bad(st->loss_sum, 8) ||
      bad(st->scratch, 16))
    return HG_ERR_INVALID_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);

  const uint64_t need = hashgrid_bwd_workspace_bytes(hg, B);
  const bool sorted = need != 0 && workspace && hashgrid_bwd_ws_pays(hg, B);
  if (sorted && (workspace_bytes < need || bad(workspace, 256))) return HG_ERR_INVALID_ARG;
  bool counted = false;
  hg_status rc = HG_ERR_UNSUPPORTED;
  if (sorted) {
    rc = hashgrid_encode_fwd_ws(hg, B, x, st->tables_half, y, workspace, workspace_bytes, stream);
    counted = rc == HG_OK;
  }
  if (rc == HG_ERR_UNSUPPORTED) rc = hashgrid_encode_fwd(hg, B, x, st->tables_half, y, stream);
  if (rc != HG_OK) return rc;

  const uint32_t n1 = 64 * n_in, n2 = 64 * 64;
  const _Float16* W = static_cast<const _Float16*>(st->weights_half);
  hg::SideJob job{};
  rc = hg::launch_mlp_train(B, n_in, n_out, y, W, W + n1, W + n1 + n2, target, st->loss, st->loss_scale, dLdy, &job,
                            st->scratch, s);
  if (rc != HG_OK) return rc;
  job.a = hg::adam_args(st->weights_adam, step);
  job.w = hg::AdamState{st->weights, static_cast<_Float16*>(st->weights_half), st->weights_m, st->weights_v};
  job.loss_sum = st->loss_sum;
  const hg::AdamArgs a = hg::adam_args(st->tables_adam, step);
  const hg::AdamState tab{st->tables, static_cast<_Float16*>(st->tables_half), st->tables_m, st->tables_v};
  if (sorted) return hg::launch_binned_adam(hg, B, x, dLdy, st->tables_zeros, workspace, counted, a, tab, job, s);
  rc = hashgrid_encode_bwd(hg, B, x, dLdy, st->tables_zeros, stream);
  return rc != HG_OK ? rc : hg::launch_adam_touched(hg, B, x, st->tables_zeros, a, tab, job, s);
}
