// Backward pass of the paper's small network (Section 4, "Architecture": two hidden layers of 64
// neurons, ReLU, linear output layer) on the matrix cores: from the encoded features y and the
// upstream gradient dL/dout to dL/dy (which hashgrid_encode_bwd[_ws] then takes to the tables) and
// the gradients of the three weight matrices, in one kernel.  Hidden activations are recomputed
// from y (they never existed in memory: the forward kernel keeps them in registers), so nothing but y
// has to be kept from the forward pass.
//
// Work unit: one wave and 32 points.  Activations and gradients of a block never leave the wave's
// registers; LDS holds the weights only.  The products, and how results
// of one are operands of the next without leaving their lanes, are in mlp_device.hpp.
// Two layouts of a matrix z[point][neuron] of a block follow:
//   "P": lane = point c, registers = neurons 32 T + 8 q + 4 h + t of tile T.  It is the B operand of
//        W z (A = rows of the weights from LDS), whose result is again in layout P: the chain
//        y -> h1 -> h2 and dL/dout -> g2 -> g1 -> dL/dy runs P to P.
//   "N": lane = neuron 32 T + c, registers = points 8 q + 4 h + t: what the weight gradients contract
//        over (the points): dW[m][n] = sum_p g[p][m] z[p][n] takes g in layout N as A and z in layout N
//        as B.  Layout N of a tile is its layout P times the identity with the operands exchanged (z as
//        A, the identity's fragment as B): the transposed result, every sum a single term, so exact.
// So a layer costs its products, one rounding of its result, and two more instructions per tile for
// the second layout; the weight gradients need no memory operand at all.  Weight-gradient sums stay
// in registers while the wave walks its blocks of points, are then added up across the workgroup's
// waves in LDS and leave with one atomic add per scalar and workgroup (training: as they are, for a later kernel).
//
// The same kernel is the network's whole part of a training step (MlpMode::kTrainL2, kTrainMape): the output layer's
// product comes out in layout P, which is where the gradient of the loss is wanted, so prediction, loss and its
// slope exist in registers only.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "hashgrid.h"
#include "hashgrid_internal.hpp"
#include "adam_device.hpp"
#include "loss_device.hpp"
#include "mlp_device.hpp"

namespace hg {

constexpr int kWaves = 4;     // waves of a workgroup: one per SIMD, which leaves a wave all 512 registers
// Blocks of 32 points a wave has in flight: two, and one where two with their targets do not fit a wave's 512 registers.
constexpr int blocks_in_flight(int KB, int OS, bool train) { return train && (KB == 2 || OS > 2) ? 1 : 2; }

enum class MlpMode {
  kBackward,   // dL/dout given: dL/dy and the weight gradients
  kTrainL2,    // targets given: the output layer and the loss between forward and backward
  kTrainMape
};

struct MlpBwdShape {
  int n_in, n_out;
  int kin_pad;   // n_in rounded up to 32: columns of the staged W1 (zero beyond n_in), rows of its transposed copy
  int out_pad;   // n_out rounded up to 16: columns of the transposed W3
  int w1_stride, w3t_stride;
  // offsets in halves from the start of LDS
  int o_w1, o_w2, o_w2t, o_w1t, o_w3t, o_w3, o_end;
  __host__ __device__ static MlpBwdShape make(int n_in, int n_out, bool train) {
    MlpBwdShape s;
    s.n_in = n_in;
    s.n_out = n_out;
    s.kin_pad = (n_in + 31) / 32 * 32;
    s.out_pad = (n_out + 15) / 16 * 16;
    s.w1_stride = s.kin_pad + kPad;
    s.w3t_stride = s.out_pad + kPad;
    s.o_w1 = 0;
    s.o_w2 = s.o_w1 + kHid * s.w1_stride;
    s.o_w2t = s.o_w2 + kHid * kHidStride;
    s.o_w1t = s.o_w2t + kHid * kHidStride;
    s.o_w3t = s.o_w1t + s.kin_pad * kHidStride;
    s.o_w3 = s.o_w3t + kHid * s.w3t_stride;  // training: W3 as it is too, 32 rows (zero from n_out on)
    s.o_end = (s.o_w3 + (train ? 32 * kHidStride : 0) + 7) / 8 * 8;
    return s;
  }
  // the weights; afterwards the same memory takes the waves' weight-gradient sums, quads (SumLayout) of 64 lanes per
  // wave, all of them at a time where they fit 128 KiB
  __host__ __device__ size_t lds_bytes(int waves) const {
    const int quads = 16 + kin_pad / 4 + 2 * ((n_out + 7) / 8);
    const size_t weights = (size_t)o_end * 2, sums = (size_t)waves * quads_per_turn(quads) * 1024;
    return weights > sums ? weights : sums;
  }
  __host__ __device__ static constexpr int quads_per_turn(int quads) { return quads <= 32 ? quads : (quads + 1) / 2; }
};

// KB: 32-column blocks of y (1 for up to 32 encoded features, else 2); OS: groups of eight outputs.
// dout: dL/dout, or the targets in the training modes; scale, loss_parts (one value per workgroup) and sums (the
// workgroups' weight-gradient sums, instead of dW1, dW2, dW3) are theirs.
template <int KB, int OS, MlpMode MODE>
__global__ __launch_bounds__(64 * kWaves) void mlp_bwd_kernel(const uint32_t B, const MlpBwdShape sh,
                                                      const _Float16* __restrict__ y, const _Float16* __restrict__ W1,
                                                      const _Float16* __restrict__ W2, const _Float16* __restrict__ W3,
                                                      const float* __restrict__ dout, _Float16* __restrict__ dy,
                                                      float* __restrict__ dW1, float* __restrict__ dW2,
                                                      float* __restrict__ dW3, const float scale,
                                                      double* __restrict__ loss_parts, float4* __restrict__ sums) {
  constexpr bool TRAIN = MODE == MlpMode::kTrainL2 || MODE == MlpMode::kTrainMape;
  constexpr int SUB = blocks_in_flight(KB, OS, TRAIN);
  constexpr int LOSS = MODE == MlpMode::kTrainL2 ? HG_LOSS_L2 : HG_LOSS_MAPE;
  extern __shared__ _Float16 lds[];
  const int n_in = sh.n_in, n_out = sh.n_out;
  const int threads = (int)blockDim.x, waves = threads / 64, wave = (int)threadIdx.x / 64, lane = (int)threadIdx.x & 63;
  _Float16* w1 = lds + sh.o_w1;    // [64][kin_pad]     W1[n][k], zero columns beyond n_in
  _Float16* w2 = lds + sh.o_w2;    // [64][64]          W2[m][n]
  _Float16* w2t = lds + sh.o_w2t;  // [64][64]          W2[m][n] at [n][m]
  _Float16* w1t = lds + sh.o_w1t;  // [kin_pad][64]     W1[n][k] at [k][n], zero rows beyond n_in
  _Float16* w3t = lds + sh.o_w3t;  // [64][out_pad]     W3[o][n] at [n][o], zero columns beyond n_out
  _Float16* w3 = lds + sh.o_w3;    // TRAIN: [32][64]   W3[o][n], zero rows from n_out on
  const int c = lane & 31, h = lane >> 5;
  constexpr uint32_t kRound = SUB * kPts;  // points of a wave's round
  const uint32_t n_rounds = (B + kRound - 1) / kRound;
  const uint32_t stride = gridDim.x * waves;
  uint32_t rnd = blockIdx.x * waves + wave;
  // y and dL/dout of a block in layout P, as they come from memory (lane = point, two pieces of four
  // encoded features or outputs per step; points beyond the batch and columns beyond n_in / n_out:
  // zeros, which add nothing).  No branches: a point beyond the batch reads the last point's row, a
  // column beyond the row its last columns, and the value is replaced by zero.
  // A wave works on SUB blocks of 32 points at a time: their chains of products do not depend on
  // each other, so the matrix cores run one block's products while the vector unit rounds the other's.
  uint2 y_next[SUB][4 * KB];
  float d_next[SUB][OS][4];
  auto request = [&](const uint64_t p0) {
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
      const uint64_t p = p0 + kPts * u + c;
      const bool inside = p < B;
      const uint64_t pr = inside ? p : (uint64_t)B - 1;
#pragma unroll
      for (int ks = 0; ks < 4 * KB; ++ks) {
        const int k = 8 * ks + 4 * h;
        const uint2 v = *reinterpret_cast<const uint2*>(y + pr * n_in + (k < n_in ? k : n_in - 4));
        const bool keep = inside && k < n_in;
        y_next[u][ks] = uint2{keep ? v.x : 0u, keep ? v.y : 0u};
      }
#pragma unroll
      for (int ks = 0; ks < OS; ++ks)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int o = 8 * ks + 4 * h + t;
          const float v = dout[pr * n_out + (o < n_out ? o : n_out - 1)];
          d_next[u][ks][t] = (inside && o < n_out) ? v : 0.0f;
        }
    }
  };

  request((uint64_t)rnd * kRound);  // the first round's, under the staging of the weights (beyond the batch: all zeros)

  // staging in pieces of four halves where the arrays allow 8-byte loads (every row length here is a multiple of 8 halves)
  const bool wide = ((reinterpret_cast<uintptr_t>(W1) | reinterpret_cast<uintptr_t>(W2) | reinterpret_cast<uintptr_t>(W3)) & 7) == 0;
  auto piece = [&](const _Float16* src, const bool inside) {
    half4 v = {(_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f};
    if (inside) {
      if (wide) {  // uniform
        v = *reinterpret_cast<const half4*>(src);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = src[t];
      }
    }
    return v;
  };
  constexpr int kThreads = 64 * kWaves;
#pragma unroll
  for (int j = 0; j < kHid * kHid / 4 / kThreads; ++j) {  // W2: 1024 pieces
    const int i = (int)threadIdx.x + j * kThreads, m = i / (kHid / 4), n = 4 * (i % (kHid / 4));
    const half4 v = piece(W2 + 4 * i, true);
    *reinterpret_cast<half4*>(w2 + m * kHidStride + n) = v;
#pragma unroll
    for (int t = 0; t < 4; ++t) w2t[(n + t) * kHidStride + m] = v[t];
  }
  for (int i = threadIdx.x; i < kHid * sh.kin_pad / 4; i += kThreads) {  // W1, zero columns beyond n_in
    const int n = i / (sh.kin_pad / 4), k = 4 * (i % (sh.kin_pad / 4));
    const half4 v = piece(W1 + n * n_in + k, k < n_in);
    *reinterpret_cast<half4*>(w1 + n * sh.w1_stride + k) = v;
#pragma unroll
    for (int t = 0; t < 4; ++t) w1t[(k + t) * kHidStride + n] = v[t];
  }
  for (int i = threadIdx.x; i < sh.out_pad * (kHid / 4); i += kThreads) {  // W3, zero columns beyond n_out
    const int o = i / (kHid / 4), n = 4 * (i % (kHid / 4));
    const half4 v = piece(W3 + o * kHid + n, o < n_out);
#pragma unroll
    for (int t = 0; t < 4; ++t) w3t[(n + t) * sh.w3t_stride + o] = v[t];
  }
  if constexpr (TRAIN) {
    for (int i = threadIdx.x; i < 32 * (kHid / 4); i += kThreads) {
      const int o = i / (kHid / 4), n = 4 * (i % (kHid / 4));
      *reinterpret_cast<half4*>(w3 + o * kHidStride + n) = piece(W3 + o * kHid + n, o < n_out);
    }
  }
  __syncthreads();

  constexpr int OJ = (OS + 1) / 2;  // steps of 16 outputs
  float16v aW2[4], aW1[2 * KB], aW3[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) aW2[i] = zero16();
#pragma unroll
  for (int i = 0; i < 2 * KB; ++i) aW1[i] = zero16();
#pragma unroll
  for (int i = 0; i < 2; ++i) aW3[i] = zero16();

  double loss_sum = 0.0;  // TRAIN: this lane's loss values

  // the identity's fragments for the exchange of y and dL/dout (step j, slot s: row 16 j + 8 (s / 4) + 4 h + s % 4, column c)
  half8 one[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int s8 = 0; s8 < 8; ++s8) one[j][s8] = (16 * j + 8 * (s8 / 4) + 4 * h + s8 % 4 == c) ? (_Float16)1.0f : (_Float16)0.0f;

  // SUB blocks of 32 points from p0 on.  FULL: all of them are inside the batch; otherwise dL/dy of the
  // points beyond it is not stored.
  auto blocks = [&](const uint64_t p0, const uint64_t p0_next, auto full) {
    constexpr bool FULL = decltype(full)::value;
    // these blocks' y and dL/dout (layout P) were requested one round ahead; request the next ones
    half8 yP[SUB][2 * KB], g3P[SUB][OJ];
    [[maybe_unused]] float target[SUB][OS][4];
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
#pragma unroll
      for (int j = 0; j < 2 * KB; ++j)
        yP[u][j] = __builtin_bit_cast(
            half8, uint4{y_next[u][2 * j].x, y_next[u][2 * j].y, y_next[u][2 * j + 1].x, y_next[u][2 * j + 1].y});
      if constexpr (TRAIN) {
#pragma unroll
        for (int ks = 0; ks < OS; ++ks)
#pragma unroll
          for (int t = 0; t < 4; ++t) target[u][ks][t] = d_next[u][ks][t];
      } else {
#pragma unroll
        for (int j = 0; j < OJ; ++j)
#pragma unroll
          for (int s8 = 0; s8 < 8; ++s8)  // rounded to half
            g3P[u][j][s8] = (2 * j + s8 / 4 < OS) ? (_Float16)d_next[u][(2 * j + s8 / 4) % OS][s8 % 4] : (_Float16)0.0f;
      }
    }
    request(p0_next);
    // layout N of one 32-column tile of a matrix in layout P (steps z[0], z[1] of the tile): z x identity
    // with the operands exchanged; every sum has one term, so the copy is exact
    auto exchange = [&](const half8* z, const int steps, half8* out) {
      float16v aN = zero16();
#pragma unroll
      for (int j = 0; j < 2; ++j)
        if (j < steps) aN = mfma(z[j], one[j], aN);
#pragma unroll
      for (int j = 0; j < 2; ++j) out[j] = to_half(aN, j);
    };
    // forward: h1 = relu(W1 y), h2 = relu(W2 h1) ([2 T + j]: tile T, step j)
    half8 h1P[SUB][4], h1N[SUB][4], h2P[SUB][4], h2N[SUB][4];
#pragma unroll
    for (int T = 0; T < 2; ++T) {
      float16v aP[SUB];
#pragma unroll
      for (int u = 0; u < SUB; ++u) aP[u] = zero16();
#pragma unroll
      for (int j = 0; j < 2 * KB; ++j) {
        const half8 w = weight_frag(w1, sh.w1_stride, T, j);
#pragma unroll
        for (int u = 0; u < SUB; ++u) aP[u] = mfma(w, yP[u][j], aP[u]);
      }
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
#pragma unroll
        for (int j = 0; j < 2; ++j) h1P[u][2 * T + j] = relu(to_half(aP[u], j));
        exchange(&h1P[u][2 * T], 2, &h1N[u][2 * T]);
      }
    }
#pragma unroll
    for (int T = 0; T < 2; ++T) {
      float16v aP[SUB];
#pragma unroll
      for (int u = 0; u < SUB; ++u) aP[u] = zero16();
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const half8 w = weight_frag(w2, kHidStride, T, j);
#pragma unroll
        for (int u = 0; u < SUB; ++u) aP[u] = mfma(w, h1P[u][j], aP[u]);
      }
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
#pragma unroll
        for (int j = 0; j < 2; ++j) h2P[u][2 * T + j] = relu(to_half(aP[u], j));
        exchange(&h2P[u][2 * T], 2, &h2N[u][2 * T]);
      }
    }
    if constexpr (TRAIN) {
      // the prediction W3 h2 in layout P (lane = point, registers = outputs 8 q + 4 h + t), and the loss's slope there
      float16v o[SUB];
#pragma unroll
      for (int u = 0; u < SUB; ++u) o[u] = zero16();
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const half8 w = weight_frag(w3, kHidStride, 0, j);
#pragma unroll
        for (int u = 0; u < SUB; ++u) o[u] = mfma(w, h2P[u][j], o[u]);
      }
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        const bool inside = FULL || p0 + kPts * u + c < B;
#pragma unroll
        for (int j = 0; j < OJ; ++j)
#pragma unroll
          for (int s8 = 0; s8 < 8; ++s8) {
            const int q = 2 * j + s8 / 4, t = s8 % 4;
            float slope = 0.0f, value = 0.0f;
            if (q < OS) {
              loss_scalar<LOSS>(o[u][4 * q + t], target[u][q % OS][t], scale, slope, value);
              if (!(inside && 8 * q + 4 * h + t < n_out)) slope = value = 0.0f;
            }
            loss_sum += (double)value;
            g3P[u][j][s8] = (_Float16)slope;  // rounded to half
          }
      }
    }
    // dL/dout in layout N (lane = output, registers = points)
    half8 g3N[SUB][2];
#pragma unroll
    for (int u = 0; u < SUB; ++u) exchange(g3P[u], OJ, g3N[u]);
    // output layer: dW3[o][n] += sum_p dout[p][o] h2[p][n];  g2 = (W3^T dout) through the ReLU of layer 2
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int T = 0; T < 2; ++T)
#pragma unroll
        for (int j = 0; j < 2; ++j) aW3[T] = mfma(g3N[u][j], h2N[u][2 * T + j], aW3[T]);
    half8 g2P[SUB][4], g2N[SUB][4];
#pragma unroll
    for (int T = 0; T < 2; ++T) {
      float16v aP[SUB];
#pragma unroll
      for (int u = 0; u < SUB; ++u) aP[u] = zero16();
#pragma unroll
      for (int j = 0; j < OJ; ++j) {
        const half8 w = weight_frag(w3t, sh.w3t_stride, T, j);
#pragma unroll
        for (int u = 0; u < SUB; ++u) aP[u] = mfma(w, g3P[u][j], aP[u]);
      }
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
#pragma unroll
        for (int j = 0; j < 2; ++j) g2P[u][2 * T + j] = where_positive(to_half(aP[u], j), h2P[u][2 * T + j]);
        exchange(&g2P[u][2 * T], 2, &g2N[u][2 * T]);
      }
    }
    // second layer: dW2[m][n] += sum_p g2[p][m] h1[p][n];  g1 = (W2^T g2) through the ReLU of layer 1
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int Tm = 0; Tm < 2; ++Tm)
#pragma unroll
        for (int Tn = 0; Tn < 2; ++Tn)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            aW2[2 * Tm + Tn] = mfma(g2N[u][2 * Tm + j], h1N[u][2 * Tn + j], aW2[2 * Tm + Tn]);
    half8 g1P[SUB][4], g1N[SUB][4];
#pragma unroll
    for (int T = 0; T < 2; ++T) {
      float16v aP[SUB];
#pragma unroll
      for (int u = 0; u < SUB; ++u) aP[u] = zero16();
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const half8 w = weight_frag(w2t, kHidStride, T, j);
#pragma unroll
        for (int u = 0; u < SUB; ++u) aP[u] = mfma(w, g2P[u][j], aP[u]);
      }
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
#pragma unroll
        for (int j = 0; j < 2; ++j) g1P[u][2 * T + j] = where_positive(to_half(aP[u], j), h1P[u][2 * T + j]);
        exchange(&g1P[u][2 * T], 2, &g1N[u][2 * T]);
      }
    }
    // first layer: dW1[n][k] += sum_p g1[p][n] y[p][k]
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int Tk = 0; Tk < KB; ++Tk) {
        half8 yN[2];
        exchange(&yP[u][2 * Tk], 2, yN);
#pragma unroll
        for (int Tn = 0; Tn < 2; ++Tn)
#pragma unroll
          for (int j = 0; j < 2; ++j) aW1[KB * Tn + Tk] = mfma(g1N[u][2 * Tn + j], yN[j], aW1[KB * Tn + Tk]);
      }
    // dL/dy = W1^T g1, layout P: four features per register group, straight to memory
#pragma unroll
    for (int Tk = 0; Tk < KB; ++Tk) {
      float16v d[SUB];
#pragma unroll
      for (int u = 0; u < SUB; ++u) d[u] = zero16();
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const half8 w = weight_frag(w1t, kHidStride, Tk, j);
#pragma unroll
        for (int u = 0; u < SUB; ++u) d[u] = mfma(w, g1P[u][j], d[u]);
      }
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        const uint64_t p = p0 + kPts * u + c;
        if (FULL || p < B) {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const half8 v = to_half(d[u], j);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const int k = 32 * Tk + 16 * j + 8 * e + 4 * h;
              if (k < n_in)  // n_in is a multiple of 8: four at once
                *reinterpret_cast<half4*>(dy + p * n_in + k) = e == 0 ? __builtin_shufflevector(v, v, 0, 1, 2, 3)
                                                                     : __builtin_shufflevector(v, v, 4, 5, 6, 7);
            }
          }
        }
      }
    }
  };

  for (; rnd < n_rounds; rnd += stride) {
    // (keeps the compiler from holding the weight fragments, which do not change from round to round, in registers)
    asm volatile("" ::: "memory");
    const uint64_t p0 = (uint64_t)rnd * kRound, p0_next = ((uint64_t)rnd + stride) * kRound;
    if (p0 + kRound <= B) blocks(p0, p0_next, std::true_type{});
    else blocks(p0, p0_next, std::false_type{});
  }

  if constexpr (TRAIN) {  // the workgroup's loss values: lanes, then waves; whoever runs next adds the workgroups up
    double* wave_sum = reinterpret_cast<double*>(lds);
    __syncthreads();  // every wave is done with the weights
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) loss_sum += __shfl_down(loss_sum, o, 64);
    if (lane == 0) wave_sum[wave] = loss_sum;
    __syncthreads();
    if (threadIdx.x == 0) {
      double total = 0.0;
      for (int w = 0; w < waves; ++w) total += wave_sum[w];
      loss_parts[blockIdx.x] = total;
    }
  }

  // The weight gradients of the workgroup.  Every wave writes its sums to LDS as they lie in its registers
  // ([wave][quad][lane], 16 bytes a lane; the weights are no longer needed), then every wave adds up all waves'
  // values of every fourth quad.  In training they leave as they are for the kernel that applies them (SideJob);
  // else with one atomic add per scalar and workgroup, workgroups starting at different quads, so that at any time
  // they add to different lines.
  float4* red = reinterpret_cast<float4*>(lds);
  constexpr int kQuads = 16 + 8 * KB + 2 * OS, kTurn = MlpBwdShape::quads_per_turn(kQuads);
  const SumLayout layout{KB, OS, n_in, n_out};
  const int rot = (int)((blockIdx.x * 5u) % (uint32_t)kTurn);
#pragma unroll
  for (int q0 = 0; q0 < kQuads; q0 += kTurn) {
    const int n_q = kQuads - q0 < kTurn ? kQuads - q0 : kTurn;
    __syncthreads();  // the area is free: every wave is done with the weights, or with the turn before
#pragma unroll
    for (int i = q0; i < q0 + n_q; ++i) {
      const float16v& acc = i < 16 ? aW2[i / 4] : i < 16 + 8 * KB ? aW1[(i - 16) / 4] : aW3[(i - 16 - 8 * KB) / OS];
      const int r = 4 * (i < 16 + 8 * KB ? i % 4 : (i - 16 - 8 * KB) % OS);
      red[(wave * kTurn + i - q0) * 64 + lane] = make_float4(acc[r], acc[r + 1], acc[r + 2], acc[r + 3]);
    }
    __syncthreads();
#pragma unroll 2
    for (int i = wave; i < n_q; i += kWaves) {
      int j = i;
      if constexpr (!TRAIN) {
        j += rot;
        j = j < n_q ? j : j - n_q;
      }
      float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float4 o = red[(w * kTurn + j) * 64 + lane];
        v[0] += o.x;
        v[1] += o.y;
        v[2] += o.z;
        v[3] += o.w;
      }
      if constexpr (TRAIN) {
        sums[((uint64_t)blockIdx.x * kQuads + q0 + j) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int k = layout.scalar_of(q0 + j, t, lane), n1 = kHid * n_in, n2 = n1 + kHid * kHid;
          if (k < 0 || v[t] == 0.0f) continue;
          float* to = k < n1 ? dW1 + k : k < n2 ? dW2 + (k - n1) : dW3 + (k - n2);
          __hip_atomic_fetch_add(to, v[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
  }
}

// The launch behind the entry points; `dout` are the targets in the training modes (loss_parts: kMaxMlpGroups doubles).
// Returns the number of workgroups through n_groups.
template <MlpMode MODE>
static hg_status launch_mlp_back(uint32_t B, uint32_t n_in, uint32_t n_out, const void* y, const void* W1, const void* W2,
                                 const void* W3, const float* dout, void* dLdy, float* dW1, float* dW2, float* dW3,
                                 float scale, double* loss_parts, float4* sums, uint32_t* n_groups, hipStream_t s) {
  constexpr bool TRAIN = MODE == MlpMode::kTrainL2 || MODE == MlpMode::kTrainMape;
  const MlpBwdShape sh = MlpBwdShape::make((int)n_in, (int)n_out, TRAIN);
  constexpr size_t kLdsLimit = 160 * 1024;
  const int waves = kWaves;
  if (sh.lds_bytes(waves) > kLdsLimit) return HG_ERR_UNSUPPORTED;
  using Kernel = void (*)(uint32_t, MlpBwdShape, const _Float16*, const _Float16*, const _Float16*, const _Float16*,
                          const float*, _Float16*, float*, float*, float*, float, double*, float4*);
  static const Kernel kernels[2][4] = {
      {mlp_bwd_kernel<1, 1, MODE>, mlp_bwd_kernel<1, 2, MODE>, mlp_bwd_kernel<1, 3, MODE>, mlp_bwd_kernel<1, 4, MODE>},
      {mlp_bwd_kernel<2, 1, MODE>, mlp_bwd_kernel<2, 2, MODE>, mlp_bwd_kernel<2, 3, MODE>, mlp_bwd_kernel<2, 4, MODE>}};
  static const hipError_t lds_ok = [] {
    hipError_t e = hipSuccess;
    for (int i = 0; i < 2 && e == hipSuccess; ++i)
      for (int j = 0; j < 4 && e == hipSuccess; ++j)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernels[i][j]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)kLdsLimit);
    return e;
  }();
  if (lds_ok != hipSuccess) return HG_ERR_DEVICE;
  // one workgroup per compute unit of the device, at most
  const uint32_t cus = cu_count() < kMaxMlpGroups ? cu_count() : kMaxMlpGroups;
  const uint32_t per_round = blocks_in_flight(sh.kin_pad / 32, (int)(n_out + 7) / 8, TRAIN) * kPts;
  const uint32_t n_rounds = (B + per_round - 1) / per_round;
  const uint32_t want = (n_rounds + waves - 1) / waves;
  const dim3 grid(want < cus ? want : cus), block(64 * waves);
  if (n_groups) *n_groups = grid.x;
  hipLaunchKernelGGL(kernels[sh.kin_pad / 32 - 1][(n_out + 7) / 8 - 1], grid, block, sh.lds_bytes(waves), s, B, sh,
                     static_cast<const _Float16*>(y), static_cast<const _Float16*>(W1), static_cast<const _Float16*>(W2),
                     static_cast<const _Float16*>(W3), dout, static_cast<_Float16*>(dLdy), dW1, dW2, dW3, scale, loss_parts,
                     sums);
  return hipGetLastError() == hipSuccess ? HG_OK : HG_ERR_DEVICE;
}

hg_status launch_mlp_train(uint32_t B, uint32_t n_in, uint32_t n_out, const void* y, const void* W1, const void* W2,
                           const void* W3, const float* target, uint32_t loss, float scale, void* dLdy, SideJob* job,
                           void* scratch, hipStream_t s) {
  double* loss_parts = static_cast<double*>(scratch);
  float4* sums = reinterpret_cast<float4*>(loss_parts + kMaxMlpGroups);
  job->at = SumLayout{(int)(n_in + 31) / 32, (int)(n_out + 7) / 8, (int)n_in, (int)n_out};
  job->blocks = (uint32_t)job->at.quads();
  job->sums = sums;
  job->loss_parts = loss_parts;
  return loss == HG_LOSS_L2
             ? launch_mlp_back<MlpMode::kTrainL2>(B, n_in, n_out, y, W1, W2, W3, target, dLdy, nullptr, nullptr, nullptr,
                                                  scale, loss_parts, sums, &job->n_parts, s)
             : launch_mlp_back<MlpMode::kTrainMape>(B, n_in, n_out, y, W1, W2, W3, target, dLdy, nullptr, nullptr, nullptr,
                                                    scale, loss_parts, sums, &job->n_parts, s);
}

}  // namespace hg

extern "C" hg_status hashgrid_mlp_bwd(uint32_t B, uint32_t n_in, uint32_t n_out, const void* y, const void* W1,
                                      const void* W2, const void* W3, const float* dLdout, void* dLdy, float* dW1,
                                      float* dW2, float* dW3, void* stream) {
  if (B == 0) return HG_OK;
  if (B > HG_MAX_BATCH) return HG_ERR_UNSUPPORTED;
  if (!y || !W1 || !W2 || !W3 || !dLdout || !dLdy || !dW1 || !dW2 || !dW3 || n_out == 0 || n_in == 0)
    return HG_ERR_INVALID_ARG;
  if (n_in % 8 != 0 || n_in > 64 || n_out > 32) return HG_ERR_UNSUPPORTED;
  auto bad = [](const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; };
  if (bad(y, 16) || bad(dLdy, 8) || bad(W1, 2) || bad(W2, 2) || bad(W3, 2) || bad(dLdout, 4) || bad(dW1, 4) ||
      bad(dW2, 4) || bad(dW3, 4))
    return HG_ERR_INVALID_ARG;
  return hg::launch_mlp_back<hg::MlpMode::kBackward>(B, n_in, n_out, y, W1, W2, W3, dLdout, dLdy, dW1, dW2, dW3, 1.0f,
                                                     nullptr, nullptr, nullptr, static_cast<hipStream_t>(stream));
}
