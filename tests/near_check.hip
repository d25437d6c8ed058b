// Compiled for the host by tests/test_host_near_pairs.py: the records that the count and scatter kernels make of a point where
// a pair's record carries both indices (plans with BinPlan::corner_records), read back as the accumulate kernel reads them.
#include <math.h>
#include <stdint.h>

#include "bwd_bins.hpp"
#include "bwd_record.hpp"
#include "hashgrid_internal.hpp"

namespace {

// Every corner's entry must receive its interpolation weight (2^-19 of it, no other entry anything), inside its chunk, and
// both passes must see the same number of records.  out[0]: violations, out[1]: pairs, out[2]: pairs that take two records.
template <int D>
void check(const hashgrid* h, uint32_t B, const float* x, uint64_t* out) {
  const hg::LevelTable& lv = h->lv;
  const hg::BinPlan& bp = h->bp;
  const bool smooth = h->cfg.interp == HG_INTERP_SMOOTHSTEP;
  const uint32_t cl = bp.chunk_log2, cmask = (1u << cl) - 1u;
  using Rec = hg::Record<float, 1>;
  const float one[1] = {1.0f};
  for (uint32_t b = 0; b < B; ++b) {
    float xp[D];
    for (int i = 0; i < D; ++i) xp[i] = x[(uint64_t)b * D + i];
    for (uint32_t l = 0; l < lv.L; ++l) {
      hg::CornerRows<D> cr, cc;
      hg::corner_rows_of<D, false>(lv, bp, l, smooth, xp, cr);
      hg::corner_rows_of<D, true>(lv, bp, l, smooth, xp, cc);  // what the count pass sees
      for (uint32_t r = 0; r < (1u << (D - 1)); ++r) {
        const uint32_t lo = 2 * r, up = 2 * r + 1;
        const hg::NearPair np = cr.pair[r];
        const bool near = np.step != hg::NearPair::kNone;
        out[0] += near != (cc.pair[r].step != hg::NearPair::kNone);
        out[1] += 1;
        out[2] += !near;
        uint32_t la, lb;
        float wl, wu;
        bool single;
        double G[1];
        if (near) {
          Rec::unpack_near(Rec::make_near(cr.la[lo], np.step, np.fraction, cr.wrow[r], one), cmask, 1.0, la, lb, wl, wu, single, G);
          if (smooth) {
            wl = hg::smoothstep(wl);
            wu = hg::smoothstep(wu);
          }
          const uint64_t e0 = (uint64_t)(cr.bin[lo] - bp.bin_base[l]) << cl;
          out[0] += cr.bin[lo] != cr.bin[up] || la != cr.la[lo] || lb != cr.la[up] || e0 + la >= lv.size[l] || e0 + lb >= lv.size[l];
          out[0] += single;
          out[0] += fabs(wl * G[0] - cr.weight[lo]) > 0x1p-19 * cr.weight[lo] || fabs(wu * G[0] - cr.weight[up]) > 0x1p-19 * cr.weight[up];
        } else {
          for (uint32_t m = lo; m <= up; ++m) {
            Rec::unpack_near(Rec::make_near(cr.la[m], hg::NearPair::kSingle, 0u, cr.weight[m], one), cmask, 1.0, la, lb, wl, wu, single, G);
            out[0] += !single || la != cr.la[m] || lb > cmask || wu != 0.0f || wl != 1.0f;
            out[0] += fabs(G[0] - cr.weight[m]) > 0x1p-19 * cr.weight[m];
          }
        }
      }
    }
  }
}

}  // namespace

extern "C" int near_check(const hashgrid_config* cfg, uint32_t B, const float* x, uint64_t* out) {
  out[0] = out[1] = out[2] = 0;
  hashgrid* h = nullptr;
  if (hashgrid_create(cfg, &h) != HG_OK) return 1;
  const bool served = h->bp.supported && h->bp.corner_records;
  if (served) cfg->d == 3 ? check<3>(h, B, x, out) : cfg->d == 2 ? check<2>(h, B, x, out) : check<1>(h, B, x, out);
  hashgrid_destroy(h);
  return served ? 0 : 1;
}
