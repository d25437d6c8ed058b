// The record of the sorted backward pass (what bin_scatter writes and bin_accumulate reads) and the
// fixed-point product of the accumulate pass.  Header-only and also compiled for the host, where
// tests check the format and its rounding without a GPU.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hg {

constexpr int kBufferWord3 = 0x00020000;  // last word of a buffer's descriptor: 32-bit elements, no swizzle

// A weight in [0,1] as a small float: `MBITS` mantissa bits under a 6-bit exponent, 0 for weights
// below 2^(LOW-127) (LOW is the fp32 exponent field that exponent code 1 stands for; such weights,
// 2^-62 and less, are far below what the fixed-point sums resolve).  The interpolation weights
// multiply dL/dy, so what the gradient needs of them is relative precision: half a unit of the
// mantissa, 2^-(MBITS+1), whatever the size of the weight.
template <int MBITS, int LOW>
__host__ __device__ __forceinline__ uint32_t pack_weight(float w) {
  const uint32_t b = __builtin_bit_cast(uint32_t, w) + (1u << (22 - MBITS));  // round to MBITS mantissa bits
  const uint32_t e8 = b >> 23;
  return e8 < (uint32_t)LOW ? 0u : ((e8 - (LOW - 1)) << MBITS) | ((b >> (23 - MBITS)) & ((1u << MBITS) - 1u));
}
template <int MBITS, int LOW>
__host__ __device__ __forceinline__ float unpack_weight(uint32_t c) {
  // exponent code and mantissa sit in the float's own order: one shift and one add rebuild it
  const uint32_t bits = (c << (23 - MBITS)) + ((uint32_t)(LOW - 1) << 23);
  return c >> MBITS ? __builtin_bit_cast(float, bits) : 0.0f;
}
constexpr uint32_t kFirstVoxel = 15u;  // value of the record's k field for a pair in the first voxel along dimension 0

// The pair of corners of a plan with BinPlan::corner_records (a table size that is no power of two, or d = 1).  Eq. 4's mod T
// comes after the XOR there, so the upper corner's entry does not follow from the lower one's and the record carries the
// difference of the two indices: the difference before the mod is +-(an odd number of k + 1 bits), k being the trailing
// one bits of the lower corner's coordinate c, and it stays that unless one of the two wraps.  The room for it is in the fraction: from c >= 2^k - 1 on
// the scaled coordinate is a multiple of 2^(k - 24), so the field of 23 bits has k - 1 low bits that are zero.  With
// |difference| = 2 e + 1 and s = number of bits of e (s <= k), the 4-bit field holds s and the sign, e's bits below its highest
// lie in the fraction's s - 1 low ones.  What does not fit that form (corners in two chunks, a wrapped index, more than 8 bits, 8 bits
// downwards, a fraction that is finer than 2^-23 as in the first voxel) is written as a record for each of the two corners (kSingle), its
// whole weight in the weight's field and the fraction 0: as exact as the pair.
// T = 1000003: 0.4 to 0.6 % of a hashed level's pairs take two records, up to 4 % at resolution 16, 1 % of all over 16 levels to 2048.
struct NearPair {
  uint32_t step;      // s, and 8 for a negative difference; kNone: the corners get a record each
  uint32_t fraction;  // fractional position along dimension 0 in units of 2^-23, e's lower bits in it
  static constexpr uint32_t kNone = 16u, kSingle = 15u;
};
// local indices la, lb in one chunk (`same`), wf the fractional position along dimension 0
__host__ __device__ __forceinline__ NearPair near_pair(const uint32_t la, const uint32_t lb, const bool same, const float wf) {
  const float q = wf * 0x1p23f;  // exact
  const bool in_field = q > 0.0f && q < 0x1p23f;
  const uint32_t q0 = in_field ? (uint32_t)q : 0u;
  const int32_t d = (int32_t)(lb - la);
  const uint32_t a = (uint32_t)(d < 0 ? -d : d);
  const uint32_t s = 31u - (uint32_t)__builtin_clz(a | 1u), low = ((1u << s) - 1u) >> 1;
  const uint32_t step = s | (d < 0 ? 8u : 0u);
  const bool fits = same && (a & 1u) && s <= 7u && step != NearPair::kSingle && (float)q0 == q && (q0 & low) == 0u;
  NearPair p;
  p.step = fits ? step : NearPair::kNone;
  p.fraction = q0 | ((a >> 1) & low);
  return p;
}

// One record = one pair of corners that differ along dimension 0, both inside one chunk.
// (Plans with BinPlan::corner_records use the other form of the header, NearPair below.)
// Two header words, then the level's F values of dL/dy as they came (fp16 pairs share a word):
//   bits 0-11   la, chunk-local index of the lower corner;
//   bits 12-15  k: on a hashed level the upper corner is lb = la ^ (2^(k+1) - 1), k = number of
//               trailing one bits of the lower corner's coordinate along dimension 0 (pi_1 = 1
//               in Eq. 4, so stepping that coordinate XORs the index with this mask, cut to the
//               table size when the table is smaller than a chunk); on a 1:1 level lb = la + 1, and k is the
//               number of trailing one bits of la, which makes it the same XOR.
//               k = 15 (kFirstVoxel) says that this coordinate is 0 (so k is 0) and that the
//               next field is in its second form;
//   bits 16-40  wrow, product of the weights of the other dimensions, as a small float (19
//               mantissa bits; 0 and 1 exact);
//   bits 41-63  the fractional position wf0 along dimension 0.  Whenever the scaled coordinate is 1
//               or more, its fraction is a multiple of 2^-23 and the field holds it exactly, in
//               units of 2^-23: both weights of the pair, wf0 and 1 - wf0, are exact.  In the first
//               voxel (scaled coordinate below 1, k = 15) the fraction can be any float: the field
//               then holds the smaller of wf0 and 1 - wf0 as a small float (16 mantissa bits) and,
//               in its top bit, which of the two that is; the other weight is 1 minus it
//               (for the smoothstep variant: of S(wf0) and S(1 - wf0) = 1 - S(wf0)).
// The reader takes the fields apart in one or two instructions each (unpack_products): the fraction is what a shift leaves of the
// second word, the weight lies across the two words where one funnel shift puts it into a double's upper half.
// 12 bytes at F = 2 with fp16 dL/dy.  A corner's summand weight * dL/dy therefore moves by at most
// 2^-20 of itself through wrow, and by 2^-17 more for a pair in the first voxel: relative
// precision, inside the 1e-5 the gradient is held to.
// The two passes over the records are bound by memory bandwidth: their size is what sets the time.
template <typename IT, int F>
struct Record {
  static constexpr uint32_t kPayloadWords = (F * sizeof(IT) + 3) / 4;
  static constexpr uint32_t kWords = 2 + kPayloadWords;
  struct Stored {
    uint32_t w[kWords];
  };
  static __host__ __device__ __forceinline__ void put_header(Stored& r, uint32_t low16, uint32_t q, float wrow) {
    const uint64_t p = (uint64_t)low16 | ((uint64_t)pack_weight<19, 65>(wrow) << 16) | ((uint64_t)q << 41);
    r.w[0] = (uint32_t)p;
    r.w[1] = (uint32_t)(p >> 32);
  }
  // the weight's 25 bits (the bits above them belong to the fraction)
  static __host__ __device__ __forceinline__ uint32_t weight_code(const Stored& r) {
    return (uint32_t)(((uint64_t)r.w[0] | ((uint64_t)r.w[1] << 32)) >> 16) & 0x1ffffffu;
  }
  // `smooth`: the smoothstep variant (Appendix A of the paper).  Only the first-voxel form needs to
  // know: it stores the pair's final weights S(wf0), S(1 - wf0), because S would double the relative
  // error of a rounded small fraction; everywhere else the fraction is exact and S is applied by the reader.
  static __host__ __device__ __forceinline__ Stored make(uint32_t la, uint32_t k, float wf0, float wrow, const IT (&g)[F],
                                                         bool smooth = false) {
    uint32_t q0;
    if (k == kFirstVoxel) {
      const float one_minus = 1.0f - wf0;
      const float up = smooth ? wf0 * wf0 * (3.0f - 2.0f * wf0) : wf0;
      const float lo = smooth ? one_minus * one_minus * (3.0f - 2.0f * one_minus) : one_minus;
      const bool upper_small = up <= lo;                // which of the pair's two weights the field holds
      q0 = (upper_small ? 0u : 1u << 22) | pack_weight<16, 64>(upper_small ? up : lo);
    } else {
      q0 = (uint32_t)rintf(wf0 * 0x1p23f);
      q0 = q0 < 0x7fffffu ? q0 : 0x7fffffu;
    }
    Stored r;
    put_header(r, la | (k << 12), q0, wrow);
    IT pay[kPayloadWords * 4 / sizeof(IT)];
#pragma unroll
    for (uint32_t f = 0; f < kPayloadWords * 4 / sizeof(IT); ++f) pay[f] = f < (uint32_t)F ? g[f] : (IT)0;
    __builtin_memcpy(&r.w[2], pay, kPayloadWords * 4);
    return r;
  }
  // NearPair's form; step = kSingle, fraction = 0 and wrow = the corner's whole weight for a record of one corner
  static __host__ __device__ __forceinline__ Stored make_near(uint32_t la, uint32_t step, uint32_t fraction, float wrow,
                                                              const IT (&g)[F]) {
    Stored r;
    put_header(r, la | (step << 12), fraction, wrow);
    IT pay[kPayloadWords * 4 / sizeof(IT)];
#pragma unroll
    for (uint32_t f = 0; f < kPayloadWords * 4 / sizeof(IT); ++f) pay[f] = f < (uint32_t)F ? g[f] : (IT)0;
    __builtin_memcpy(&r.w[2], pay, kPayloadWords * 4);
    return r;
  }
  // la, lb, weights and totals as unpack_scaled gives them; single: the record is one corner's (w_up is 0 and lb names no
  // entry of its own)
  static __host__ __device__ __forceinline__ void unpack_near(const Stored& r, uint32_t cmask, double scale, uint32_t& la,
                                                              uint32_t& lb, float& w_lo, float& w_up, bool& single,
                                                              double (&G)[F]) {
    la = r.w[0] & 0xfffu & cmask;
    single = ((r.w[0] >> 12) & 15u) == NearPair::kSingle;
    const uint32_t s = (r.w[0] >> 12) & 7u, q = r.w[1] >> 9, low = q & (((1u << s) - 1u) >> 1);
    const uint32_t a = (1u << s) | (low << 1) | 1u;
    lb = (r.w[0] & 0x8000u ? la - a : la + a) & cmask;
    w_up = (float)(q - low) * 0x1p-23f;
    w_lo = 1.0f - w_up;  // exact
    const double wrow = (double)unpack_weight<19, 65>(weight_code(r)) * scale;
    IT pay[kPayloadWords * 4 / sizeof(IT)];
    __builtin_memcpy(pay, &r.w[2], kPayloadWords * 4);
#pragma unroll
    for (int f = 0; f < F; ++f) G[f] = wrow * (double)(float)pay[f];
  }
  // a record at `offset` bytes of a buffer; zeros beyond its end.  The whole offset is in the operand that the buffer's bound is sure
  // to cover: the compiler's documentation leaves the load's scalar offset out of the bounds check.
  static __device__ __forceinline__ Stored load_from(__amdgpu_buffer_rsrc_t buffer, uint32_t offset) {
    typedef uint32_t words2 __attribute__((ext_vector_type(2)));
    typedef uint32_t words3 __attribute__((ext_vector_type(3)));
    typedef uint32_t words4 __attribute__((ext_vector_type(4)));
    constexpr int kStream = 2;  // read once
    Stored r;
    uint32_t q = 0;
#pragma unroll
    for (; q + 4 <= kWords; q += 4) {
      const words4 v = __builtin_amdgcn_raw_buffer_load_b128(buffer, offset + 4 * q, 0, kStream);
      __builtin_memcpy(&r.w[q], &v, 16);
    }
    if constexpr (kWords % 4 == 3) {
      const words3 v = __builtin_amdgcn_raw_buffer_load_b96(buffer, offset + 4 * q, 0, kStream);
      __builtin_memcpy(&r.w[q], &v, 12);
    } else if constexpr (kWords % 4 == 2) {
      const words2 v = __builtin_amdgcn_raw_buffer_load_b64(buffer, offset + 4 * q, 0, kStream);
      __builtin_memcpy(&r.w[q], &v, 8);
    }
    return r;
  }
  static __host__ __device__ __forceinline__ Stored load(const uint32_t* base, uint32_t i) {
    const uint32_t* p = base + (uint64_t)i * kWords;
    Stored r;
#pragma unroll
    for (uint32_t q = 0; q < kWords; ++q) r.w[q] = __builtin_nontemporal_load(p + q);
    return r;
  }
  // la, lb, the pair's two weights along dimension 0 (w_lo for the lower corner, w_up for the upper
  // one: 1 - wf0 and wf0, to which the reader applies the smoothstep where the variant asks for it,
  // unless `first` says that the record is in its first-voxel form, which holds the final weights)
  // and the F totals of the pair, wrow * dL/dy_f, as doubles times `scale`: a 20-bit by at most
  // 24-bit product, exact in a double.
  // `xmask`: on a hashed level, the chunk's entry count minus one (a table smaller than a chunk
  // wraps the XOR); `cmask`: the chunk capacity minus one
  static __host__ __device__ __forceinline__ void unpack_scaled(const Stored& r, bool dense, uint32_t cmask, uint32_t xmask,
                                                       double scale, uint32_t& la, uint32_t& lb, float& w_lo,
                                                       float& w_up, bool& first, double (&G)[F]) {
    la = r.w[0] & 0xfffu & cmask;
    uint32_t k = (r.w[0] >> 12) & 0xfu;
    const uint32_t q0 = r.w[1] >> 9;
    first = k == kFirstVoxel;
    if (__builtin_expect(first, 0)) {  // rare: one voxel in N_l along dimension 0
      k = 0;
      const float small = unpack_weight<16, 64>(q0 & 0x3fffffu), big = 1.0f - small;
      const bool upper_small = (q0 >> 22) == 0u;
      w_up = upper_small ? small : big;
      w_lo = upper_small ? big : small;
    } else {
      w_up = (float)q0 * 0x1p-23f;
      w_lo = 1.0f - w_up;  // exact
    }
    lb = dense ? (la + 1u) & cmask : la ^ (((2u << k) - 1u) & xmask);
    const double wrow = (double)unpack_weight<19, 65>(weight_code(r)) * scale;
    IT pay[kPayloadWords * 4 / sizeof(IT)];
    __builtin_memcpy(pay, &r.w[2], kPayloadWords * 4);
#pragma unroll
    for (int f = 0; f < F; ++f) G[f] = wrow * (double)(float)pay[f];
  }
  // What the accumulate pass multiplies and where it adds: byte offsets of the two entries' 64-bit sums (la8, lb8) and, as
  // doubles, the weights along dimension 0 and the totals times a power of two, so that w * G is
  // weight * wrow * dL/dy * 2^S exactly, as with unpack_scaled.  About 30 vector instructions a record of two features with the
  // additions, half of what the conversions through single precision and a branch for 1:1 levels came to; the pass
  // spends more time on them than on the additions in LDS.
  //   without smoothstep the weights are the fraction's integer and 2^23 minus it, and exponent = S - 23; with it exponent = S;
  //   the double of wrow is its code with the exponent moved: a code of 0 reads as 2^(S - 63) (or 2^(S - 86)) instead of 0, whose
  //   products round to 0 (|dL/dy| 2^S <= 2^51);
  //   xmask: chunk capacity minus 1 on a 1:1 level.
  template <bool SMOOTH, bool NEAR>
  static __host__ __device__ __forceinline__ void unpack_products(const Stored& r, bool dense, uint32_t cmask, uint32_t xmask,
                                                                  int exponent, uint32_t& la8, uint32_t& lb8, double& w_lo,
                                                                  double& w_up, double (&G)[F]) {
    const uint32_t w0 = r.w[0], w1 = r.w[1], cmask8 = cmask << 3, xmask8 = xmask << 3;
    la8 = (w0 << 3) & cmask8;
    uint32_t q = w1 >> 9;
    if (NEAR) {
      const uint32_t s = (w0 >> 12) & 7u, low = q & (((1u << s) - 1u) >> 1);
      const uint32_t a8 = (8u << s) | (low << 4) | 8u;
      lb8 = (w0 & 0x8000u ? la8 - a8 : la8 + a8) & cmask8;
      q -= low;
    } else {
      lb8 = la8 ^ (((16u << ((w0 >> 12) & 15u)) - 8u) & xmask8);
    }
    if (SMOOTH) {
      const float up = (float)q * 0x1p-23f, lo = 1.0f - up;
      w_up = (double)(up * up * (3.0f - 2.0f * up));
      w_lo = (double)(lo * lo * (3.0f - 2.0f * lo));
    } else {
      w_up = (double)q;
      w_lo = 0x1p23 - w_up;
    }
    if (!NEAR && __builtin_expect((w0 & 0xf000u) == kFirstVoxel << 12, 0)) {  // rare: one voxel in N_l along dimension 0
      lb8 = dense ? (la8 + 8u) & cmask8 : la8 ^ (8u & xmask8);
      const float small = unpack_weight<16, 64>(q & 0x3fffffu), big = 1.0f - small;
      const bool upper_small = (q >> 22) == 0u;
      w_up = (double)(upper_small ? small : big) * (SMOOTH ? 1.0 : 0x1p23);
      w_lo = (double)(upper_small ? big : small) * (SMOOTH ? 1.0 : 0x1p23);
    }
    const uint32_t code2 = (uint32_t)(((uint64_t)w0 | ((uint64_t)w1 << 32)) >> 15) & 0x3fffffeu;  // (19 mantissa bits in a place for 20)
    const double wrow = __builtin_bit_cast(double, (uint64_t)(code2 + ((uint32_t)(960 + exponent) << 20)) << 32);
    IT pay[kPayloadWords * 4 / sizeof(IT)];
    __builtin_memcpy(pay, &r.w[2], kPayloadWords * 4);
#pragma unroll
    for (int f = 0; f < F; ++f) G[f] = wrow * (double)(float)pay[f];
  }
};

// round(w * G) to a 64-bit integer (ties to even), for |w * G| < 2^51: adding
// 1.5 * 2^52 leaves the integer, in two's complement, in the low bits of the
// double.  One rounding, of the exact product.
constexpr int kFixedBits = 51;
__host__ __device__ __forceinline__ unsigned long long fixed_product(double w, double G) {
  const double d = __builtin_fma(w, G, 0x1.8p52);
  return (unsigned long long)(__builtin_bit_cast(long long, d) - __builtin_bit_cast(long long, 0x1.8p52));
}

}  // namespace hg
