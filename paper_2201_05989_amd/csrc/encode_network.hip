// The encoding followed by the small network of the paper (Section 4, "Architecture": two hidden
// layers of 64 neurons, ReLU, linear output layer): the output at a batch of points, and its gradient with respect to
// the position.  The encoded features go from the gathers into LDS rows, from there into the matrix
// cores' operand registers, and through the layers without leaving them (mlp_device.hpp); nothing between the
// table entries and the result reaches memory unless the caller keeps the features for training.
//
// Two shapes.  `encode_network` is one thread per point, level after level, for batches that fill the chip; its workgroups
// stage the weights once and walk the batch.  `encode_network_split` gives a block of 64 points to eight waves, each wave every eighth
// level: for small batches, where a thread that walks all the levels is one long chain of gather latencies
// (13 us for any batch up to a few thousand points, of which the split kernel needs 4).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>

#include "hashgrid.h"
#include "hashgrid_common.hpp"
#include "hashgrid_internal.hpp"
#include "mlp_device.hpp"

namespace hg {

constexpr int kMaxOut = 32;  // output neurons (one 32-row block of the matrix instruction)
constexpr int kOutStride = kMaxOut + kPad;

// The weights in LDS, rows padded by kPad halves: w1 [64][n_in up to a multiple of 32, zeros beyond n_in], w2 [64][64],
// w3 [32][64] (zero rows from n_out on); for the way back, instead of w3, the transposed ones: w3t [64][32] (zero columns
// from n_out on), w2t [64][64], w1t [n_in up to a multiple of 32][64] (zero rows beyond n_in).  What a product contracts
// over, and the rows that become the next product's operand, are in the order of place16.
struct NetShape {
  int n_in, n_out, k32;
  int w1_stride;
  int o_w2, o_w3, o_w3t, o_w2t, o_w1t, o_end;  // offsets in halves; w1 at 0
  __host__ __device__ static NetShape make(int n_in, int n_out, bool back) {
    NetShape s;
    s.n_in = n_in;
    s.n_out = n_out;
    s.k32 = (n_in + 31) / 32 * 32;
    s.w1_stride = s.k32 + kPad;
    s.o_w2 = kHid * s.w1_stride;
    s.o_w3 = s.o_w2 + kHid * kHidStride;
    s.o_w3t = s.o_w3 + (back ? 0 : kMaxOut * kHidStride);
    s.o_w2t = s.o_w3t + (back ? kHid * kOutStride : 0);
    s.o_w1t = s.o_w2t + (back ? kHid * kHidStride : 0);
    s.o_end = s.o_w1t + (back ? s.k32 * kHidStride : 0);
    return s;
  }
};

// BACK: what the gradient needs (W1, W2 both ways, W3 transposed); else the three layers.  The arrays are 8-byte aligned.
template <bool BACK>
__device__ __forceinline__ void stage_weights(_Float16* lds, const NetShape& sh, const _Float16* __restrict__ W1,
                                              const _Float16* __restrict__ W2, const _Float16* __restrict__ W3) {
  const int block = (int)blockDim.x;
  const half4 zero = {(_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f};
  const int q1 = sh.k32 / 4;
  for (int i = threadIdx.x; i < kHid * q1; i += block) {
    const int n = i / q1, k = 4 * (i % q1);
    const half4 v = k < sh.n_in ? *reinterpret_cast<const half4*>(W1 + n * sh.n_in + k) : zero;
    *reinterpret_cast<half4*>(lds + place16(n) * sh.w1_stride + place16(k)) = v;
    if (BACK) {
#pragma unroll
      for (int t = 0; t < 4; ++t) lds[sh.o_w1t + (k + t) * kHidStride + place16(n)] = v[t];
    }
  }
  constexpr int q2 = kHid / 4;
  for (int i = threadIdx.x; i < kHid * q2; i += block) {
    const int m = i / q2, n = 4 * (i % q2);
    const half4 v = *reinterpret_cast<const half4*>(W2 + 4 * i);
    *reinterpret_cast<half4*>(lds + sh.o_w2 + place16(m) * kHidStride + place16(n)) = v;
    if (BACK) {
#pragma unroll
      for (int t = 0; t < 4; ++t) lds[sh.o_w2t + (place16(n) + t) * kHidStride + place16(m)] = v[t];
    }
  }
  for (int i = threadIdx.x; i < kMaxOut * q2; i += block) {
    const int o = i / q2, n = 4 * (i % q2);
    const half4 v = o < sh.n_out ? *reinterpret_cast<const half4*>(W3 + 4 * i) : zero;
    if (BACK) {
#pragma unroll
      for (int t = 0; t < 4; ++t) lds[sh.o_w3t + (place16(n) + t) * kOutStride + place16(o)] = v[t];
    } else {
      *reinterpret_cast<half4*>(lds + sh.o_w3 + o * kHidStride + place16(n)) = v;
    }
  }
}

// Rows of encoded features in LDS: n_in halves and kPad of padding, 8-byte aligned
__device__ __forceinline__ int row_stride(const NetShape& sh) { return sh.n_in + kPad; }

// A level's features of a point into its row.  A feature is the fp32 sum, rounded to half: left alone the compiler makes one
// instruction with one rounding (v_fma_mixlo_f16) of the last multiply-add and the conversion in some kernels and not in
// others, and a feature that the forward call keeps is then now and then not the one that the way back has.  KEEP holds the
// sums as they are.  In the split kernel eight features, and two where a wave has four levels, come out so by themselves, and
// holding them there costs registers that the kernel does not have (77000 points, 8 levels of 8, there and back: 38 us, 63 with what it spills).
// (F = 1: the one instruction in all of them, the forward kernel included.)
template <int F, bool KEEP>
__device__ __forceinline__ void put_features(float (&acc)[F], _Float16* at) {
  if constexpr (!KEEP) {
#pragma unroll
    for (int f = 0; f < F; ++f) at[f] = (_Float16)acc[f];
  } else {
#pragma unroll
    for (int f = 0; f < F; ++f) asm("" : "+v"(acc[f]));
    _Float16* to = static_cast<_Float16*>(__builtin_assume_aligned(at, 2 * F));
#pragma unroll
    for (int f = 0; f < F; f += 2) {
      const half2v h = __builtin_convertvector((float2v{acc[f], acc[f + 1]}), half2v);
      to[f] = h[0];
      to[f + 1] = h[1];
    }
  }
}

// A lane's part of the features of 16 points as an operand: `row` is its point's row (lane % 16), in LDS or memory, 8-byte aligned; g = lane / 16
__device__ __forceinline__ void load_features(const _Float16* row, const NetShape& sh, const int g, half8 (&y)[2]) {
  const half4 zero = {(_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (32 * j >= sh.n_in) break;  // uniform
    const int k0 = 32 * j + 16 * (g / 2) + 4 * (g % 2), k1 = k0 + 8;  // (a column beyond the row reads its first ones, and is replaced by zero)
    const half4 lo = *reinterpret_cast<const half4*>(row + (k0 < sh.n_in ? k0 : 0));
    const half4 hi = *reinterpret_cast<const half4*>(row + (k1 < sh.n_in ? k1 : 0));
    y[j] = __builtin_shufflevector(k0 < sh.n_in ? lo : zero, k1 < sh.n_in ? hi : zero, 0, 1, 2, 3, 4, 5, 6, 7);
  }
}

// Rows 16 T .. 16 T + 15 of w z for U times 16 points of the wave; steps: 32 columns each.  A weight fragment is read
// once for all of them.
template <int U>
__device__ __forceinline__ void tile(const _Float16* w, const int stride, const int T, const half8 (&z)[U][2], const int steps,
                                     float4v (&a)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) a[u] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (j >= steps) break;  // uniform
    const half8 f = weight_frag16(w, stride, T, j);
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = mfma16(f, z[u][j], a[u]);
  }
}

// One layer of 64 rows: operand z to operand out(u, j, 16-bit values of rows 32 j ..)
template <int U, typename Out>
__device__ __forceinline__ void layer(const _Float16* w, const int stride, const half8 (&z)[U][2], const int steps, Out out) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float4v lo[U], hi[U];
    tile<U>(w, stride, 2 * j, z, steps, lo);
    tile<U>(w, stride, 2 * j + 1, z, steps, hi);
#pragma unroll
    for (int u = 0; u < U; ++u) out(u, j, to_half16(lo[u], hi[u]));
    asm volatile("" ::: "memory");  // loads of weight fragments stay on their side: moved up together they would not fit the registers
  }
}

// BACK: the activations as the way back needs them (relu: zeros are +0), the network's backward pass has the same.  A NaN is 0
// to both forms, see relu.
template <int U, bool BACK>
__device__ __forceinline__ void hidden_layers(const _Float16* lds, const NetShape& sh, const half8 (&y)[U][2],
                                              half8 (&h1)[U][2], half8 (&h2)[U][2]) {
  layer<U>(lds, sh.w1_stride, y, sh.k32 / 32, [&](int u, int j, half8 v) { h1[u][j] = BACK ? relu(v) : relu_max(v); });
  layer<U>(lds + sh.o_w2, kHidStride, h1, 2, [&](int u, int j, half8 v) { h2[u][j] = BACK ? relu(v) : relu_max(v); });
}

// The network on U times 16 points of a wave, p + 16 u being this lane's (p: the first block's point of lane % 16), row[u] its row
template <int U>
__device__ __forceinline__ void network(const _Float16* lds, const NetShape& sh, const _Float16* (&row)[U], const uint64_t p,
                                        const uint32_t B, float* __restrict__ out) {
  half8 y[U][2], h1[U][2], h2[U][2];
  const int g = ((int)threadIdx.x & 63) >> 4;
#pragma unroll
  for (int u = 0; u < U; ++u) load_features(row[u], sh, g, y[u]);
  hidden_layers<U, false>(lds, sh, y, h1, h2);
#pragma unroll
  for (int T = 0; T < 2; ++T) {
    if (16 * T >= sh.n_out) break;  // uniform
    float4v o[U];
    tile<U>(lds + sh.o_w3, kHidStride, T, h2, 2, o);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float* at = out + (p + 16 * u) * (uint64_t)sh.n_out;
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (p + 16 * u < B && 16 * T + 4 * g + t < sh.n_out) at[16 * T + 4 * g + t] = o[u][t];
    }
  }
}

// The network alone, on features that are in memory (hashgrid_mlp_fwd): a wave takes 32 points at a time
constexpr int kMlpOnlyBlock = 256;
__global__ __launch_bounds__(kMlpOnlyBlock) void mlp_fwd_from_features(const uint32_t B, const NetShape sh,
                                                                       const _Float16* __restrict__ y,
                                                                       const _Float16* __restrict__ W1,
                                                                       const _Float16* __restrict__ W2,
                                                                       const _Float16* __restrict__ W3,
                                                                       float* __restrict__ out) {
  extern __shared__ _Float16 lds[];
  stage_weights<false>(lds, sh, W1, W2, W3);
  __syncthreads();
  const uint32_t c = threadIdx.x & 15;
  for (uint64_t p0 = ((uint64_t)blockIdx.x * kMlpOnlyBlock + (threadIdx.x & ~63u)) / 2; p0 < B;
       p0 += (uint64_t)gridDim.x * kMlpOnlyBlock / 2) {
    asm volatile("" ::: "memory");  // (keeps the weight fragments out of registers between rounds, here and below)
    const _Float16* row[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint64_t p = p0 + 16 * u + c;
      row[u] = y + (p < B ? p : B - 1) * sh.n_in;  // idle lanes shadow the last point
    }
    network<2>(lds, sh, row, p0 + c, B, out);
  }
}

// One thread per point, level by level, as the forward kernel (hashgrid.hip) with the gathers of later levels issued before
// a level is blended.  The levels whose gathers look ahead to a level that exists have a loop without a condition: behind one
// the compiler counts loads in flight as if the later level's were not there, and waits for them too (d = 3, 16 levels of
// one feature, T = 2^19, 33000 points in random order: 31.4 us with the condition, 25.4 without).
// PACED: a barrier per level keeps the waves of a workgroup on the same slice of the tables, as there: 2^20 points at T = 2^19,
// d = 3, take 332 us in 1024-thread workgroups with it and 625 us without.  Otherwise the waves run free and one wave's
// products run under another's gathers: 2^20 pixels of a raster at T = 2^22 75 us, 89 with the barrier.  That is for tables that
// stay in an XCD's L2 and are too wide for the L1 to gain from the order either (d = 3, F of 4 or 8: 91 against 105 us), and for
// d = 2 as long as neighbouring lanes have neighbouring points: a workgroup whose first block of points is in no such order
// (kNear) paces itself all the same, and then looks one level ahead and not three (what the three touch is more than the order keeps).
constexpr float kNear = 1.0f / 64.0f;
constexpr int kNetBlock = 1024;
template <int D, int F, bool PACED>
__global__ __launch_bounds__(kNetBlock, 4) void encode_network(
    const LevelTable lv, const bool smooth, const uint32_t B, const NetShape sh, const float* __restrict__ x,
    const _Float16* __restrict__ theta, const _Float16* __restrict__ W1, const _Float16* __restrict__ W2,
    const _Float16* __restrict__ W3, float* __restrict__ out, _Float16* __restrict__ y_out) {
  extern __shared__ _Float16 lds[];
  const int stride = row_stride(sh);
  const uint32_t block = blockDim.x;
  _Float16* rows = lds + sh.o_end;  // [block][stride]
  _Float16* my_row = rows + (int)threadIdx.x * stride;
  const uint32_t lane = threadIdx.x & 63, wave0 = threadIdx.x & ~63u;
  bool near = false;
  if constexpr (!PACED && D == 2) {
    const uint64_t i = (uint64_t)blockIdx.x * block + threadIdx.x, j = i + 1 < B ? i + 1 : B - 1;
    const float* xi = x + (i < B ? i : B - 1) * D;
    near = fabsf(xi[0] - x[j * D]) < kNear && fabsf(xi[1] - x[j * D + 1]) < kNear;
  }
  stage_weights<false>(lds, sh, W1, W2, W3);
  bool pace = PACED;
  if constexpr (!PACED && D == 2) pace = __syncthreads_count(near) < (int)block / 2;  // (the barrier behind the staging)
  else __syncthreads();
  auto walk = [&](auto pace) {
    for (uint64_t p0 = (uint64_t)blockIdx.x * block; p0 < B; p0 += (uint64_t)gridDim.x * block) {
      asm volatile("" ::: "memory");
      const uint64_t b0 = p0 + threadIdx.x;
      const uint32_t b = b0 < B ? (uint32_t)b0 : B - 1;  // idle lanes of the last block shadow the last point
      float xp[D];
#pragma unroll
      for (int i = 0; i < D; ++i) xp[i] = x[(uint64_t)b * D + i];
      constexpr int kSets = D == 2 && F <= 2 && !decltype(pace)::value ? 4 : D == 3 && F == 8 ? 1 : 2;  // register sets: kSets - 1 levels are in flight ahead
      Vec<_Float16, F> e[kSets][1 << D];
      float wr[kSets][1 << (D - 1)], w0[kSets], u0[kSets];
      auto gather_level = [&](const uint32_t l, const int set) {
        uint32_t idx[1 << D];
        level_corners<D, true>(lv, l, smooth, xp, idx, wr[set], w0[set], u0[set]);
        const Vec<_Float16, F>* tab = reinterpret_cast<const Vec<_Float16, F>*>(theta) + lv.offset[l];
#pragma unroll
        for (uint32_t m = 0; m < (1u << D); ++m) e[set][m] = tab[idx[m]];
      };
      auto blend_level = [&](const uint32_t l, const int set) {
        float acc[F];
#pragma unroll
        for (int f = 0; f < F; ++f) acc[f] = 0.0f;
#pragma unroll
        for (uint32_t m = 0; m < (1u << D); ++m) {
          const float wt = wr[set][m >> 1] * ((m & 1u) ? w0[set] : u0[set]);
#pragma unroll
          for (int f = 0; f < F; ++f) acc[f] = fmaf(wt, (float)e[set][m].v[f], acc[f]);
        }
        put_features<F, (F > 1)>(acc, my_row + l * F);
        asm volatile("" ::: "memory");  // keep the gathers of one level together
        if constexpr (decltype(pace)::value) __syncthreads();
      };
#pragma unroll
      for (int j = 0; j < kSets - 1; ++j)
        if (j < (int)lv.L) gather_level(j, j);  // uniform, here and below
      uint32_t l0 = 0;
#pragma unroll 1
      for (; l0 + 2 * kSets - 1 <= lv.L; l0 += kSets) {
#pragma unroll
        for (int j = 0; j < kSets; ++j) {
          gather_level(l0 + j + kSets - 1, (j + kSets - 1) % kSets);
          blend_level(l0 + j, j);
        }
      }
#pragma unroll 1
      for (; l0 < lv.L; l0 += kSets) {
#pragma unroll
        for (int j = 0; j < kSets; ++j) {
          const uint32_t ahead = l0 + j + kSets - 1;
          if (ahead < lv.L) gather_level(ahead, (j + kSets - 1) % kSets);
          if (l0 + j < lv.L) blend_level(l0 + j, j);
        }
      }
      // from here on a wave reads the rows of its own 64 points only
      if (y_out != nullptr) {
        // training: the encoded features as the network sees them; a wave's rows are one run of memory
        const int pieces = sh.n_in / 8;
        for (int i = (int)lane; i < 64 * pieces; i += 64) {
          const int r = i / pieces, k = 8 * (i % pieces);
          const uint64_t p = p0 + wave0 + r;
          if (p >= B) continue;
          const _Float16* at = rows + ((int)wave0 + r) * stride + k;
          const half4 lo = *reinterpret_cast<const half4*>(at), hi = *reinterpret_cast<const half4*>(at + 4);
          *reinterpret_cast<half8*>(y_out + p * sh.n_in + k) = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
      }
#pragma unroll 1
      for (int half = 0; half < 2; ++half) {
        const int r = (int)wave0 + 32 * half + (int)(lane & 15);
        const _Float16* row[2] = {rows + r * stride, rows + (r + 16) * stride};
        network<2>(lds, sh, row, p0 + r, B, out);
      }
      asm volatile("" ::: "memory");
    }
  };
  if constexpr (PACED) {
    walk(std::true_type{});
  } else if constexpr (D == 2) {
    if (pace) walk(std::true_type{});
    else walk(std::false_type{});
  } else {
    walk(std::false_type{});
  }
}

// A block of 64 points and eight waves; wave w has the levels w, w + 8, ...: LPW of them at most, all their gathers in
// flight at once.  Four of the waves then run the network, 16 points each.
// GRAD: not the output but its gradient with respect to the position.  The four waves go on from the hidden
// activations back to the gradient of the features, which all waves contract with the entries they still hold.  The levels'
// parts are added up in the order of the levels: the bits are those of the three calls that the kernel stands for.
template <int F>
__device__ __forceinline__ void keep_packed(Vec<_Float16, F>& v) {
  if constexpr (F == 1) {
    asm volatile("" : "+v"(v.v[0]));
  } else {
    uint32_t w[F / 2];
    __builtin_memcpy(w, &v, sizeof(w));
#pragma unroll
    for (int i = 0; i < F / 2; ++i) asm volatile("" : "+v"(w[i]));
    __builtin_memcpy(&v, w, sizeof(w));
  }
}

constexpr int kSplitWaves = 8, kSplitPoints = 64;
template <int D, int F, int LPW, bool GRAD>
__global__ __launch_bounds__(64 * kSplitWaves, 4) void encode_network_split(
    const LevelTable lv, const bool smooth, const uint32_t B, const NetShape sh, const float* __restrict__ x,
    const _Float16* __restrict__ theta, const _Float16* __restrict__ W1, const _Float16* __restrict__ W2,
    const _Float16* __restrict__ W3, const float* __restrict__ dout, float* __restrict__ out, _Float16* __restrict__ y_out) {
  extern __shared__ _Float16 lds[];
  const int stride = row_stride(sh);
  _Float16* rows = lds + sh.o_end;  // [kSplitPoints][stride]
  float* part = reinterpret_cast<float*>(rows + (kSplitPoints * stride + 7) / 8 * 8);  // GRAD: [L][D][kSplitPoints]
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  stage_weights<GRAD>(lds, sh, W1, W2, W3);
  for (uint64_t p0 = (uint64_t)blockIdx.x * kSplitPoints; p0 < B; p0 += (uint64_t)gridDim.x * kSplitPoints) {
    asm volatile("" ::: "memory");
    const uint64_t b0 = p0 + lane;
    const uint32_t b = b0 < B ? (uint32_t)b0 : B - 1;  // idle lanes of the last block shadow the last point
    float xp[D];
#pragma unroll
    for (int i = 0; i < D; ++i) xp[i] = x[(uint64_t)b * D + i];
    Vec<_Float16, F> e[LPW][1 << D];
    float wr[LPW][1 << (D - 1)], w0[LPW], u0[LPW];
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
      const uint32_t l = wave + kSplitWaves * q;
      if (l >= lv.L) break;  // uniform
      uint32_t idx[1 << D];
      level_corners<D, true>(lv, l, smooth, xp, idx, wr[q], w0[q], u0[q]);
      const Vec<_Float16, F>* tab = reinterpret_cast<const Vec<_Float16, F>*>(theta) + lv.offset[l];
#pragma unroll
      for (uint32_t m = 0; m < (1u << D); ++m) e[q][m] = tab[idx[m]];
    }
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
      const uint32_t l = wave + kSplitWaves * q;
      if (l >= lv.L) break;  // uniform
      float acc[F];
#pragma unroll
      for (int f = 0; f < F; ++f) acc[f] = 0.0f;
#pragma unroll
      for (uint32_t m = 0; m < (1u << D); ++m) {
        const float wt = wr[q][m >> 1] * ((m & 1u) ? w0[q] : u0[q]);
#pragma unroll
        for (int f = 0; f < F; ++f) acc[f] = fmaf(wt, (float)e[q][m].v[f], acc[f]);
      }
      put_features<F, F == 4 || (F == 2 && LPW < 4)>(acc, rows + lane * stride + l * F);
    }
    __syncthreads();  // the rows are complete (and, the first time, the weights)
    if (!GRAD && y_out != nullptr) {
      const int pieces = sh.n_in / 4;
      for (int i = (int)threadIdx.x; i < kSplitPoints * pieces; i += 64 * kSplitWaves) {
        const int r = i / pieces, k = 4 * (i % pieces);
        if (p0 + r < B)
          *reinterpret_cast<half4*>(y_out + (p0 + r) * sh.n_in + k) = *reinterpret_cast<const half4*>(rows + r * stride + k);
      }
    }
    if (wave < kSplitPoints / 16) {
      int at = lane;
      if constexpr (GRAD) asm volatile("" : "+v"(at));  // what follows from it is not kept in registers from one round to the next
      const int c = at & 15, g = at >> 4, r = 16 * wave + c;
      const uint64_t p = p0 + r;
      if constexpr (!GRAD) {
        const _Float16* row[1] = {rows + r * stride};
        network<1>(lds, sh, row, p, B, out);
      } else {
        half8 y[1][2], h1[1][2], h2[1][2], z[1][2];
        load_features(rows + r * stride, sh, g, y[0]);
        hidden_layers<1, true>(lds, sh, y, h1, h2);
        // dL/dout, rounded to half as the backward pass of the network rounds it
        const float* d = dout != nullptr ? dout + (p < B ? p : B - 1) * (uint64_t)sh.n_out : nullptr;
#pragma unroll
        for (int s8 = 0; s8 < 8; ++s8) {
          const int o = 16 * (g / 2) + 8 * (s8 / 4) + 4 * (g % 2) + s8 % 4;
          z[0][0][s8] = (_Float16)0.0f;
          if (o < sh.n_out) z[0][0][s8] = d != nullptr ? (_Float16)d[o] : (_Float16)1.0f;
        }
        // through the ReLUs: g2 = W3^T dL/dout where h2 > 0, g1 = W2^T g2 where h1 > 0
        layer<1>(lds + sh.o_w3t, kOutStride, z, 1, [&](int u, int j, half8 v) { h2[u][j] = where_positive(v, h2[u][j]); });
        layer<1>(lds + sh.o_w2t, kHidStride, h2, 2, [&](int u, int j, half8 v) { z[u][j] = where_positive(v, h1[u][j]); });
        // dL/dy = W1^T g1, rounded to half, over the features of the same points
#pragma unroll
        for (int T = 0; T < 4; ++T) {
          if (16 * T >= sh.n_in) break;  // uniform
          float4v a[1];
          tile<1>(lds + sh.o_w1t, kHidStride, T, z, 2, a);
          const half4 v = __builtin_convertvector(a[0], half4);
          if (16 * T + 4 * g < sh.n_in) *reinterpret_cast<half4*>(rows + r * stride + 16 * T + 4 * g) = v;
        }
      }
    }
    __syncthreads();  // every reader of the rows is done (GRAD: dL/dy is in them)
    if constexpr (GRAD) {
#pragma unroll
      for (int i = 0; i < D; ++i) asm volatile("" : "+v"(xp[i]));  // the weights are computed again, not kept in registers across the network,
#pragma unroll
      for (int q = 0; q < LPW; ++q) {
        const uint32_t l = wave + kSplitWaves * q;
        if (l >= lv.L) break;  // uniform
        float g[F], gx[D];
#pragma unroll
        for (int i = 0; i < D; ++i) gx[i] = 0.0f;
#pragma unroll
        for (uint32_t m = 0; m < (1u << D); ++m) keep_packed(e[q][m]);  // ... and the entries stay halves across it
#pragma unroll
        for (int f = 0; f < F; ++f) g[f] = (float)rows[lane * stride + l * F + f];
        add_position_gradient<D, F>(lv, l, smooth, xp, e[q], g, gx);
#pragma unroll
        for (int i = 0; i < D; ++i) part[(l * D + i) * kSplitPoints + lane] = gx[i];
      }
      __syncthreads();
      const int t = (int)threadIdx.x;
      if (t < kSplitPoints * D && p0 + t / D < B) {
        float sum = 0.0f;
        for (uint32_t l = 0; l < lv.L; ++l) sum += part[(l * D + t % D) * kSplitPoints + t / D];
        out[p0 * D + t] = sum;
      }
    }
  }
}

// Threads of a workgroup where two of half the size fit a compute unit: the batch spread evenly over both, as point_major_block
// spreads it over one
static uint32_t half_block(uint32_t B) {
  constexpr uint64_t kMost = kNetBlock / 2;
  const uint64_t slots = 2 * cu_count(), rounds = (B + kMost * slots - 1) / (kMost * slots);
  const uint64_t per_wg = (B + rounds * slots - 1) / (rounds * slots);
  return (uint32_t)((per_wg + 63) / 64 * 64);
}

template <int D, int F>
static hg_status launch_network(const hashgrid* h, uint32_t B, const float* x, const void* params, const void* W1,
                                const void* W2, const void* W3, uint32_t n_out, float* out, void* y_out, hipStream_t s) {
  const int n_in = (int)h->lv.L * F;
  const NetShape sh = NetShape::make(n_in, (int)n_out, false);
  const bool smooth = h->cfg.interp == HG_INTERP_SMOOTHSTEP;
  const _Float16 *t = static_cast<const _Float16*>(params), *w1 = static_cast<const _Float16*>(W1),
                 *w2 = static_cast<const _Float16*>(W2), *w3 = static_cast<const _Float16*>(W3);
  _Float16* yo = static_cast<_Float16*>(y_out);
  // The split kernel holds until the batch gives every thread of the other shape a point or so.  Its waves are at all levels at
  // once, so beyond an XCD's L2 it loses to the paced one earlier where the points are in no order, and with more than eight
  // levels, where a wave has two, earlier still: the line lies where one order wins what the other loses.  Split against not, us,
  // 16 levels of 2: d = 3, T = 2^19, 30000 points random 28.0 and 28.0, rays 17.6 and 22.4, 40000 points 37.2 and 31.1, 22.7 and
  // 24.8; T = 2^15, 50000 points 21.9 and 19.0, 14.3 and 16.7; d = 2, T = 2^19, 70000 points random 25.6 and 24.0, raster 12.6 and
  // 13.1; T = 2^15, 100000 points 17.6 and 18.2, 11.8 and 12.6.  8 levels of 8, d = 3, T = 2^19, 40000 points random 28.1 and 30.8,
  // rays 17.7 and 23.4; T = 2^15, 100000 points 25.3 and 25.3, 15.5 and 17.0.
  constexpr uint64_t kL2Bytes = 4u << 20;
  const bool large = h->total * F * sizeof(_Float16) > kL2Bytes, paced = D == 3 && (F <= 2 || large);
  const uint32_t most = h->lv.L <= kSplitWaves ? (D == 3 && large ? 40000u : 100000u)
                        : D == 3               ? (large ? 32768u : 50000u)
                                               : (large ? 70000u : 100000u);
  if (B <= most) {
    const size_t lds = ((size_t)sh.o_end + (kSplitPoints * (n_in + kPad) + 7) / 8 * 8) * sizeof(_Float16);
    const uint32_t blocks = (B + kSplitPoints - 1) / kSplitPoints, slots = 2 * cu_count();
    const dim3 grid(blocks < slots ? blocks : slots), block(64 * kSplitWaves);
#define HG_SPLIT(LPW)                                                                                                   \
  hipLaunchKernelGGL((encode_network_split<D, F, LPW, false>), grid, block, lds, s, h->lv, smooth, B, sh, x, t, w1, w2, \
                     w3, nullptr, out, yo)
    if (h->lv.L <= 8) {
      HG_SPLIT(1);
    } else if (h->lv.L <= 16) {
      if constexpr (F <= 4) HG_SPLIT(2);  // (L * F is 64 at most)
    } else {
      if constexpr (F <= 2) HG_SPLIT(4);
    }
#undef HG_SPLIT
    return hipGetLastError() == hipSuccess ? HG_OK : HG_ERR_DEVICE;
  }
  // One workgroup of up to 1024 threads a compute unit where the order of the levels counts, or where two of 512 do not fit (64
  // features: half the waves otherwise; d = 2, T = 2^19, 16 levels of 4, 2^20 points random 271 us, now 210, raster 92, now 64);
  // two of 512 else (d = 2, T = 2^15, 16 levels of 2, 2^18 points random 33 us, 35 with one).
  const bool two_fit = 2 * ((size_t)sh.o_end + (size_t)(kNetBlock / 2) * (n_in + kPad)) * sizeof(_Float16) <= 160 * 1024;
  const uint32_t block = paced || large || !two_fit ? point_major_block(B) : half_block(B);
  const size_t lds = ((size_t)sh.o_end + (size_t)block * (n_in + kPad)) * sizeof(_Float16);
  static const hipError_t lds_ok = [] {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(encode_network<D, F, false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256);  // (the vote on the order has some of its own)
    if constexpr (D == 3) {
      if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(encode_network<D, F, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    }
    return e;
  }();
  if (lds_ok != hipSuccess) return HG_ERR_DEVICE;
  const uint32_t blocks = (B + block - 1) / block, per_cu = (uint32_t)(160 * 1024 / lds),
                 slots = (per_cu < kNetBlock / block ? per_cu : kNetBlock / block) * cu_count();
  const dim3 grid(blocks < slots ? blocks : slots);
  if (paced) {
    if constexpr (D == 3)
      hipLaunchKernelGGL((encode_network<D, F, true>), grid, dim3(block), lds, s, h->lv, smooth, B, sh, x, t, w1, w2, w3, out,
                         yo);
  } else {
    hipLaunchKernelGGL((encode_network<D, F, false>), grid, dim3(block), lds, s, h->lv, smooth, B, sh, x, t, w1, w2, w3, out,
                       yo);
  }
  return hipGetLastError() == hipSuccess ? HG_OK : HG_ERR_DEVICE;
}

template <int D, int F>
static hg_status launch_network_grad(const hashgrid* h, uint32_t B, const float* x, const void* params, const void* W1,
                                     const void* W2, const void* W3, uint32_t n_out, const float* dout, float* dx,
                                     hipStream_t s) {
  const int n_in = (int)h->lv.L * F;
  const NetShape sh = NetShape::make(n_in, (int)n_out, true);
  const size_t lds = ((size_t)sh.o_end + (kSplitPoints * (n_in + kPad) + 7) / 8 * 8) * sizeof(_Float16) +
                     (size_t)h->lv.L * D * kSplitPoints * sizeof(float);  // 59 KB at most up to 16 levels, then 71
  const uint32_t blocks = (B + kSplitPoints - 1) / kSplitPoints, slots = 2 * cu_count();
  const dim3 grid(blocks < slots ? blocks : slots), block(64 * kSplitWaves);
#define HG_SPLIT(LPW)                                                                                                  \
  hipLaunchKernelGGL((encode_network_split<D, F, LPW, true>), grid, block, lds, s, h->lv,                              \
                     h->cfg.interp == HG_INTERP_SMOOTHSTEP, B, sh, x, static_cast<const _Float16*>(params),            \
                     static_cast<const _Float16*>(W1), static_cast<const _Float16*>(W2),                               \
                     static_cast<const _Float16*>(W3), dout, dx, static_cast<_Float16*>(nullptr))
  if (h->lv.L <= 8) {
    HG_SPLIT(1);
  } else if (h->lv.L <= 16) {
    if constexpr (F <= 4) HG_SPLIT(2);  // (L * F is 64 at most)
  } else {
    if constexpr (F <= 2) {
      static const hipError_t lds_ok = hipFuncSetAttribute(reinterpret_cast<const void*>(encode_network_split<D, F, 4, true>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
      if (lds_ok != hipSuccess) return HG_ERR_DEVICE;
      HG_SPLIT(4);
    }
  }
#undef HG_SPLIT
  return hipGetLastError() == hipSuccess ? HG_OK : HG_ERR_DEVICE;
}

}  // namespace hg

static bool bad_pointer(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

// what the two entry points with the encoding in front ask of their arguments
static hg_status check_network(const hashgrid_t* hg, uint32_t B, const float* x, const void* params, const void* W1,
                               const void* W2, const void* W3, uint32_t n_out, const float* out) {
  if (B > HG_MAX_BATCH) return HG_ERR_UNSUPPORTED;
  if (!x || !params || !W1 || !W2 || !W3 || !out || n_out == 0) return HG_ERR_INVALID_ARG;
  const hashgrid_config& c = hg->cfg;
  const uint32_t n_in = c.L * c.F;
  if (c.param_dtype != HG_F16 || !hg->lv.T_is_pow2 || c.d < 2 || n_in % 8 != 0 || n_in > (uint32_t)hg::kHid ||
      n_out > (uint32_t)hg::kMaxOut)
    return HG_ERR_UNSUPPORTED;
  if (bad_pointer(x, 4) || bad_pointer(params, c.F * 2) || bad_pointer(W1, 8) || bad_pointer(W2, 8) || bad_pointer(W3, 8) ||
      bad_pointer(out, 4))
    return HG_ERR_INVALID_ARG;
  return HG_OK;
}

#define HG_BY_SHAPE(c, CALL)             \
  switch ((c).d * 16 + (c).F) {          \
    case 2 * 16 + 1: return CALL(2, 1);  \
    case 2 * 16 + 2: return CALL(2, 2);  \
    case 2 * 16 + 4: return CALL(2, 4);  \
    case 2 * 16 + 8: return CALL(2, 8);  \
    case 3 * 16 + 1: return CALL(3, 1);  \
    case 3 * 16 + 2: return CALL(3, 2);  \
    case 3 * 16 + 4: return CALL(3, 4);  \
    case 3 * 16 + 8: return CALL(3, 8);  \
    default: return HG_ERR_UNSUPPORTED;  \
  }

static hg_status encode_mlp_fwd_any(const hashgrid_t* hg, uint32_t B, const float* x, const void* params, const void* W1,
                                    const void* W2, const void* W3, uint32_t n_out, float* out, void* y_out,
                                    void* stream) {
  if (!hg) return HG_ERR_INVALID_ARG;
  if (B == 0) return HG_OK;
  const hg_status ok = check_network(hg, B, x, params, W1, W2, W3, n_out, out);
  if (ok != HG_OK) return ok;
  if (bad_pointer(y_out, 16)) return HG_ERR_INVALID_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
#define HG_NET(D, F) hg::launch_network<D, F>(hg, B, x, params, W1, W2, W3, n_out, out, y_out, s)
  HG_BY_SHAPE(hg->cfg, HG_NET)
#undef HG_NET
}

extern "C" hg_status hashgrid_encode_mlp_fwd(const hashgrid_t* hg, uint32_t B, const float* x, const void* params,
                                             const void* W1, const void* W2, const void* W3, uint32_t n_out,
                                             float* out, void* stream) {
  return encode_mlp_fwd_any(hg, B, x, params, W1, W2, W3, n_out, out, nullptr, stream);
}

extern "C" hg_status hashgrid_encode_mlp_fwd_train(const hashgrid_t* hg, uint32_t B, const float* x, const void* params,
                                                   const void* W1, const void* W2, const void* W3, uint32_t n_out,
                                                   float* out, void* y, void* stream) {
  if (B != 0 && !y) return HG_ERR_INVALID_ARG;
  return encode_mlp_fwd_any(hg, B, x, params, W1, W2, W3, n_out, out, y, stream);
}

extern "C" hg_status hashgrid_encode_mlp_bwd_input(const hashgrid_t* hg, uint32_t B, const float* x, const void* params,
                                                   const void* W1, const void* W2, const void* W3, uint32_t n_out,
                                                   const float* dLdout, float* dLdx, void* stream) {
  if (!hg) return HG_ERR_INVALID_ARG;
  if (B == 0) return HG_OK;
  const hg_status ok = check_network(hg, B, x, params, W1, W2, W3, n_out, dLdx);
  if (ok != HG_OK) return ok;
  if (bad_pointer(dLdout, 4)) return HG_ERR_INVALID_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
#define HG_NET(D, F) hg::launch_network_grad<D, F>(hg, B, x, params, W1, W2, W3, n_out, dLdout, dLdx, s)
  HG_BY_SHAPE(hg->cfg, HG_NET)
#undef HG_NET
}

extern "C" hg_status hashgrid_mlp_fwd(uint32_t B, uint32_t n_in, uint32_t n_out, const void* y, const void* W1,
                                      const void* W2, const void* W3, float* out, void* stream) {
  if (B == 0) return HG_OK;
  if (B > HG_MAX_BATCH) return HG_ERR_UNSUPPORTED;
  if (!y || !W1 || !W2 || !W3 || !out || n_in == 0 || n_out == 0) return HG_ERR_INVALID_ARG;
  if (n_in % 8 != 0 || n_in > (uint32_t)hg::kHid || n_out > (uint32_t)hg::kMaxOut) return HG_ERR_UNSUPPORTED;
  if (bad_pointer(y, 16) || bad_pointer(W1, 8) || bad_pointer(W2, 8) || bad_pointer(W3, 8) || bad_pointer(out, 4))
    return HG_ERR_INVALID_ARG;
  const hg::NetShape sh = hg::NetShape::make((int)n_in, (int)n_out, false);
  const uint32_t want = (B + 127) / 128, slots = 4 * hg::cu_count();
  hipLaunchKernelGGL(hg::mlp_fwd_from_features, dim3(want < slots ? want : slots), dim3(hg::kMlpOnlyBlock),
                     (size_t)sh.o_end * sizeof(_Float16), static_cast<hipStream_t>(stream), B, sh,
                     static_cast<const _Float16*>(y), static_cast<const _Float16*>(W1),
                     static_cast<const _Float16*>(W2), static_cast<const _Float16*>(W3), out);
  return hipGetLastError() == hipSuccess ? HG_OK : HG_ERR_DEVICE;
}
