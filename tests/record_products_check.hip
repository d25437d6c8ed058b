// Compiled for the host by tests/test_host_record_products.py: what the accumulate pass's reader makes of a record
// (unpack_products) against the plain one (unpack_scaled, unpack_near).
#include <stdint.h>

#include "bwd_bins.hpp"
#include "bwd_record.hpp"

namespace {
// 1 for a record whose entries differ, or whose rounded products differ for some feature
template <typename IT, int F, bool SMOOTH, bool NEAR>
uint32_t differs(const typename hg::Record<IT, F>::Stored& r, bool dense, uint32_t cmask, uint32_t xmask, int S) {
  using Rec = hg::Record<IT, F>;
  uint32_t la, lb, la8, lb8;
  float lo, up;
  double G[F], w_lo, w_up, H[F];
  bool first;
  const double scale = __builtin_ldexp(1.0, S);
  if (NEAR) Rec::unpack_near(r, cmask, scale, la, lb, lo, up, first, G);
  else Rec::unpack_scaled(r, dense, cmask, xmask, scale, la, lb, lo, up, first, G);
  if (SMOOTH && !first) {
    lo = hg::smoothstep(lo);
    up = hg::smoothstep(up);
  }
  Rec::template unpack_products<SMOOTH, NEAR>(r, dense, cmask, dense ? cmask : xmask, SMOOTH ? S : S - 23, la8, lb8, w_lo, w_up, H);
  uint32_t bad = la8 != 8 * la || lb8 != 8 * lb;
  for (int f = 0; f < F; ++f)
    bad |= hg::fixed_product(lo, G[f]) != hg::fixed_product(w_lo, H[f]) || hg::fixed_product(up, G[f]) != hg::fixed_product(w_up, H[f]);
  return bad;
}

template <typename IT, int F, bool SMOOTH>
uint32_t check(uint32_t n, const uint32_t* la, const uint32_t* c0, const float* wf0, const float* wrow, const float* g, int dense,
               uint32_t cmask, uint32_t xmask, int S) {
  using Rec = hg::Record<IT, F>;
  uint32_t bad = 0;
  for (uint32_t i = 0; i < n; ++i) {
    IT gi[F];
    for (int f = 0; f < F; ++f) gi[f] = (IT)g[(uint64_t)i * F + f];
    hg::Rows<2> rw;
    rw.la[0] = la[i];
    rw.k = c0[i] == 0 ? hg::kFirstVoxel : (uint32_t)__builtin_ctz(~c0[i] | 0x4000u);
    bad += differs<IT, F, SMOOTH, false>(Rec::make(la[i], hg::record_k<2>(rw, 0, dense), wf0[i], wrow[i], gi, SMOOTH), dense, cmask, xmask, S);
    const uint32_t lb = la[i] ^ (((2u << (c0[i] % 5)) - 1u) & cmask);
    const hg::NearPair np = hg::near_pair(la[i], lb, true, wf0[i]);
    const bool near = np.step != hg::NearPair::kNone;
    bad += differs<IT, F, SMOOTH, true>(Rec::make_near(la[i], near ? np.step : hg::NearPair::kSingle, near ? np.fraction : 0u, wrow[i], gi),
                                        false, cmask, xmask, S);
  }
  return bad;
}
}  // namespace

// Records that differ.  c0: the lower corner's coordinate along dimension 0; S: exponent of the sums' unit
extern "C" uint32_t products_check(uint32_t F, int half, int smooth, uint32_t n, const uint32_t* la, const uint32_t* c0, const float* wf0,
                                   const float* wrow, const float* g, int dense, uint32_t cmask, uint32_t xmask, int S) {
#define HG_PC(IT, FF)                                                                     \
  (smooth ? check<IT, FF, true>(n, la, c0, wf0, wrow, g, dense, cmask, xmask, S) \
          : check<IT, FF, false>(n, la, c0, wf0, wrow, g, dense, cmask, xmask, S))
  switch (F) {
    case 1: return half ? HG_PC(_Float16, 1) : HG_PC(float, 1);
    case 2: return half ? HG_PC(_Float16, 2) : HG_PC(float, 2);
    case 4: return half ? HG_PC(_Float16, 4) : HG_PC(float, 4);
    case 8: return half ? HG_PC(_Float16, 8) : HG_PC(float, 8);
    default: return n;
  }
#undef HG_PC
}
