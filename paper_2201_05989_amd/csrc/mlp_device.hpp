// The 64-64 network's products on the matrix cores with activations in registers (paper Section 4, "Architecture"),
// shared by the kernels that run it: forward behind the encoding (encode_network.hip), backward (mlp_bwd.hip).
//
// Every product is v_mfma_f32_32x32x16_f16 (fp16 operands, fp32 accumulation), D[i][j] = sum_k A[i][k] B[k][j] over 16
// values of k, with, per lane l (c = l % 32, h = l / 32):
//   A: row i = c, eight values of k in registers;   B: column j = c, eight values of k;
//   D: column j = c, rows i = 8 q + 4 h + t in register 4 q + t (q, t = 0 .. 3).
// Which eight k a lane holds is the instruction's business only in that A and B must agree, so k is
// numbered here the way D comes out: slot s = 0 .. 7 of lane half h in step j stands for
// k = 16 j + 8 (s / 4) + 4 h + s % 4.  Then a lane's part of D, rounded to half, register groups
// 2 j and 2 j + 1, is already its part of the B (or A) operand of step j of a product that contracts
// over D's rows, and the matching fragment of a weight row is two 8-byte pieces 16 bytes apart.
// "Layout P" of a matrix z[point][neuron] of 32 points: lane = point c, registers = neurons 32 T + 8 q + 4 h + t of
// tile T.  It is the B operand of W z (A = rows of the weights from LDS), whose result is again in layout P.
//
// v_mfma_f32_16x16x32_f16 works the same way on 16 points (functions that end in 16): c = l % 16, g = l / 16, D rows
// 4 g + t in register t.  A quarter of the registers and half of the latency of a block, for twice the weight reads a
// point.  It adds the products of lane groups 0 and 1 to the accumulator and then those of 2 and 3, so its slots stand for
// what two steps of the instruction above have in theirs, k = 32 j + 16 (g / 2) + 8 (s / 4) + 4 (g % 2) + s % 4, and its
// sums are the same bits (2^16 sums of 64 random products on an MI355X: all equal; with k = 32 j + 16 (s / 4) + 4 g + s % 4
// 62 % differ in the last bit, which now and then takes a half or a ReLU the other way).  In that order D's rows are what the
// next operand needs if the weight arrays have index n of a contracted (or next) dimension at place16(n); a lane's piece of a
// row is then 32 bytes from its other one.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hashgrid.h"

namespace hg {

constexpr int kHid = 64;      // neurons of a hidden layer
constexpr int kPad = 4;       // halves of padding per LDS row: the 8-byte reads of 32 lanes a row apart cover all banks
constexpr int kHidStride = kHid + kPad;
constexpr int kPts = 32;      // points of a wave's block

using half2v = _Float16 __attribute__((ext_vector_type(2)));
using half4 = _Float16 __attribute__((ext_vector_type(4)));
using half8 = _Float16 __attribute__((ext_vector_type(8)));
using short8v = short __attribute__((ext_vector_type(8)));
using float8v = float __attribute__((ext_vector_type(8)));
using float16v = float __attribute__((ext_vector_type(16)));
using float2v = float __attribute__((ext_vector_type(2)));
using float4v = float __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float16v zero16() {
  float16v z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.0f;
  return z;
}
__device__ __forceinline__ float16v mfma(const half8 a, const half8 b, const float16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
// register groups 2 j and 2 j + 1 of a result, rounded to half (nearest even): step j of an operand
__device__ __forceinline__ half8 to_half(const float16v& acc, const int j) {
  float8v v;
#pragma unroll
  for (int s = 0; s < 8; ++s) v[s] = acc[8 * j + s];
  return __builtin_convertvector(v, half8);
}
// ReLU on halves: as 16-bit integers the negative halves (and -0) are the negative numbers.  So is a NaN that a matrix
// instruction made, the only ones that come here: it is 0xffc00000 for every pair of zeros, ones, largest, infinite and NaN
// operands of either sign, in both instructions (tried on an MI355X), and 0xfe00 as a half.
__device__ __forceinline__ half8 relu(const half8 v) {
  return __builtin_bit_cast(half8, __builtin_elementwise_max(__builtin_bit_cast(short8v, v), (short8v)0));
}
// ReLU for an output that nothing is propagated back from: max(v, 0) as the floating-point maximum has it, NaN to 0
__device__ __forceinline__ half8 relu_max(const half8 v) { return __builtin_elementwise_max(v, (half8)(_Float16)0.0f); }
// g where the activation act (not negative: it went through relu) is positive, else 0: all ones
// where the bits of act are not zero, two packed instructions for two halves (written out: the
// compiler would turn the C expression into a compare and a select per half)
__device__ __forceinline__ half8 where_positive(const half8 g, const half8 act) {
  uint4 a = __builtin_bit_cast(uint4, act);
  const uint4 gb = __builtin_bit_cast(uint4, g);
  // (op_sel_hi: the upper half of the instruction takes the shift count from the constant's lower 16 bits too)
  asm("v_pk_sub_i16 %0, 0, %0\n\tv_pk_ashrrev_i16 %0, 15, %0 op_sel_hi:[0,1]" : "+v"(a.x));
  asm("v_pk_sub_i16 %0, 0, %0\n\tv_pk_ashrrev_i16 %0, 15, %0 op_sel_hi:[0,1]" : "+v"(a.y));
  asm("v_pk_sub_i16 %0, 0, %0\n\tv_pk_ashrrev_i16 %0, 15, %0 op_sel_hi:[0,1]" : "+v"(a.z));
  asm("v_pk_sub_i16 %0, 0, %0\n\tv_pk_ashrrev_i16 %0, 15, %0 op_sel_hi:[0,1]" : "+v"(a.w));
  return __builtin_bit_cast(half8, uint4{gb.x & a.x, gb.y & a.y, gb.z & a.z, gb.w & a.w});
}

__device__ __forceinline__ float4v mfma16(const half8 a, const half8 b, const float4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
// the results of tiles 2 j and 2 j + 1 of a layer, rounded to half (nearest even): step j of an operand
__device__ __forceinline__ half8 to_half16(const float4v lo, const float4v hi) {
  return __builtin_convertvector(__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7), half8);
}
// Where a weight array has neuron (or input) n: bits 3 and 4 change places
__device__ __forceinline__ constexpr int place16(const int n) { return (n & ~24) | ((n & 8) << 1) | ((n & 16) >> 1); }
// A lane's fragment of row 16 T + c of a weight array in LDS for step j: columns 32 j + 4 g .. + 3 and 32 j + 16 + 4 g .. + 3
__device__ __forceinline__ half8 weight_frag16(const _Float16* w, const int stride, const int T, const int j) {
  const int lane = (int)threadIdx.x & 63;
  const _Float16* at = w + (16 * T + (lane & 15)) * stride + 32 * j + 4 * (lane >> 4);
  const half4 lo = *reinterpret_cast<const half4*>(at), hi = *reinterpret_cast<const half4*>(at + 16);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// A lane's fragment of row 32 T + c of a weight array in LDS for step j: columns 16 j + 4 h .. + 3 and 16 j + 8 + 4 h .. + 3
__device__ __forceinline__ half8 weight_frag(const _Float16* w, const int stride, const int T, const int j) {
  const int lane = (int)threadIdx.x & 63;
  const _Float16* at = w + (32 * T + (lane & 31)) * stride + 16 * j + 4 * (lane >> 5);
  const half4 lo = *reinterpret_cast<const half4*>(at), hi = *reinterpret_cast<const half4*>(at + 8);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

}  // namespace hg
