// Kernels of the learned coarse-lattice correction: a per-node network
// 54 -> 64 -> 64 -> 5 with exact GELU, BF16 weights and activations, FP32
// accumulation on the matrix cores (v_mfma_f32_16x16x16_bf16), its training
// step (forward, backward, weight gradients, Adam), and the lattice side:
// full-weighting restriction of a fine state onto a coarse one, the 3x3
// stencil features, the correction targets and the momentum source
// F = dJ + div(dtau) through which a correction acts on the scheme.
//
// Matrix-core layout (16x16x16, wave64, lane l = 16 g + c):
//   A (16 x 16, M x K): lane holds row c, k = 4 g .. 4 g + 3
//   B (16 x 16, K x N): lane holds column c, k = 4 g .. 4 g + 3
//   C (16 x 16, M x N): lane holds column c, rows 4 g .. 4 g + 3
// The network is evaluated transposed, Z^T = W A^T with nodes as the N
// dimension, so that a C tile of one layer (units x nodes) is, register for
// register, the B operand of the next layer.  One wave handles 16 nodes.
#include "tpl_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

namespace tplk {

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest even (finite inputs).
__device__ __forceinline__ short bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (short)(u >> 16);
}

__device__ __forceinline__ v4s pack4(const v4f &v) {
  return v4s{bf16_bits(v[0]), bf16_bits(v[1]), bf16_bits(v[2]), bf16_bits(v[3])};
}

__device__ __forceinline__ v4s ld4(const uint16_t *p) {
  return *reinterpret_cast<const v4s *>(p);
}

__device__ __forceinline__ v4f mfma(const v4s &a, const v4s &b, const v4f &c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

constexpr float kInvSqrt2 = 0.70710678118654752f;
constexpr float kInvSqrt2Pi = 0.39894228040143268f;

// exact GELU z Phi(z)
__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * kInvSqrt2)); }
// and with it its derivative Phi(z) + z phi(z), from the same erf
__device__ __forceinline__ float gelu_grad(float z, float &grad) {
  const float e = 1.0f + erff(z * kInvSqrt2);
  grad = 0.5f * e + z * kInvSqrt2Pi * expf(-0.5f * z * z);
  return 0.5f * z * e;
}

// Forward pass of one 16-node tile (nodes n0 .. n0 + 15, lane column c).
// Outputs z3 (standardised outputs 4 g + i); keeps the GELU's derivatives d1,
// d2 at the pre-activations and the BF16 operands x, h1, h2 for the backward
// pass.
struct Tile {
  v4s x[4];    // input, B operand per K-block
  v4f d1[4], d2[4];
  v4s h1[4], h2[4];
  v4f z3;
};

// The three layers from the input operands already in t.x (GRAD: with the
// derivatives).
template <bool GRAD>
__device__ __forceinline__ void tile_layers(const MlpDev &w, int c, int g, Tile &t) {
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) {
    v4f acc;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = w.b1[16 * mb + 4 * g + i];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
      acc = mfma(ld4(w.W1b + (16 * mb + c) * 64 + 16 * kb + 4 * g), t.x[kb], acc);
    v4f h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float d = 0.0f;
      h[i] = GRAD ? gelu_grad(acc[i], d) : gelu(acc[i]);
      t.d1[mb][i] = d;
    }
    t.h1[mb] = pack4(h);
  }
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) {
    v4f acc;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = w.b2[16 * mb + 4 * g + i];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
      acc = mfma(ld4(w.W2b + (16 * mb + c) * 64 + 16 * kb + 4 * g), t.h1[kb], acc);
    v4f h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float d = 0.0f;
      h[i] = GRAD ? gelu_grad(acc[i], d) : gelu(acc[i]);
      t.d2[mb][i] = d;
    }
    t.h2[mb] = pack4(h);
  }
  v4f acc;
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = w.b3[4 * g + i];
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) acc = mfma(ld4(w.W3b + c * 64 + 16 * kb + 4 * g), t.h2[kb], acc);
  t.z3 = acc;
}

// Standardisation of the inputs a lane feeds: inputs 16 kb + 4 g + i.
struct InNorm {
  float mean[4][4], stdv[4][4];
};
__device__ __forceinline__ void load_norm(const float *__restrict__ mean,
                                          const float *__restrict__ stdv, int nin, int g,
                                          InNorm &w) {
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = 16 * kb + 4 * g + i;
      w.mean[kb][i] = k < nin ? mean[k] : 0.0f;
      w.stdv[kb][i] = k < nin ? stdv[k] : 1.0f;
    }
}

// The input operands of a tile straight from the raw FP32 rows X [n][nin]:
// standardised, rounded to BF16, zero beyond the inputs and the nodes.
__device__ __forceinline__ void tile_inputs(const InNorm &w, const float *__restrict__ X,
                                            long long n, int nin, long long node, int g, Tile &t) {
  const bool valid = node < n;
  const float *row = X + node * nin;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    v4s v = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = 16 * kb + 4 * g + i;
      if (valid && k < nin) v[i] = bf16_bits((row[k] - w.mean[kb][i]) / w.stdv[kb][i]);
    }
    t.x[kb] = v;
  }
}

}  // namespace

// Y[n][nout] = network(standardised X) mapped back to physical units.
__global__ void __launch_bounds__(256)
    k_mlp_forward(MlpDev w, const float *__restrict__ mean, const float *__restrict__ stdv,
                  const float *__restrict__ X, long long n, float *__restrict__ Y) {
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const long long n0 = ((long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 16;
  if (n0 >= n) return;  // whole wave
  const long long node = n0 + c;
  InNorm nm;
  load_norm(mean, stdv, w.nin, g, nm);
  Tile t;
  tile_inputs(nm, X, n, w.nin, node, g, t);
  tile_layers<false>(w, c, g, t);
  if (node < n)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = 4 * g + i;
      if (o < w.nout) Y[node * w.nout + o] = t.z3[i] * w.out_std[o] + w.out_mean[o];
    }
}

// Training pass: a workgroup of eight waves walks chunks of 128 nodes, one
// 16-node tile per wave.  Each wave runs forward and backward on its tile and
// stages the operands of the weight gradients transposed (units x the chunk's
// 128 nodes, BF16) in the workgroup's LDS; the 36 16 x 16 blocks of dW1, dW2
// and dW3 are then shared out over the waves, each contracted over all 128
// nodes.  Gradients of loss = mean over nodes and outputs of (y - t)^2
// (standardised targets) go to the workgroup's record in partial[]:
//   dW1 [64][64] | db1 [64] | dW2 [64][64] | db2 [64] | dW3 [16][64] |
//   db3 [16] | sum of squared errors [1]         (kMlpRecord doubles)
//
// Sums over nodes are FP32 inside the matrix cores and FP64 from run to run
// (a finished run is added to the record in memory: the registers cannot hold
// FP64 blocks).  A run is never longer than the share of one of 512 waves that
// walk the tiles alone: RUN tiles of a chunk, or with RUN = 0 `chunks` chunks.
//
// What bounds it: the vector ALUs (32 erf and 32 exp per lane and tile against
// 92 matrix instructions), so every SIMD should have two waves; a wave that
// holds all 36 blocks (144 accumulators) and walks tiles alone leaves one wave
// on every second SIMD.  65536 rows: 108 us that way, with a launch before it
// that wrote the standardised inputs (10 us), against 66 here (58 with sums in
// FP32 over all of a workgroup's chunks).
constexpr int kTrainWaves = 8, kTrainNodes = 16 * kTrainWaves;
constexpr int kTrainStride = kTrainNodes + 8;  // LDS rows: 16 units of a read fall in 16 bank groups
template <int RUN>
__global__ void __launch_bounds__(64 * kTrainWaves)
    k_mlp_train(MlpDev w, const float *__restrict__ mean, const float *__restrict__ stdv,
                const float *__restrict__ X, const float *__restrict__ T, long long n, float scale,
                int chunks, double *__restrict__ partial) {
  // rows: X 0, H1 64, H2 128, dZ1 192, dZ2 256, dY 320
  __shared__ __align__(16) uint16_t st[336][kTrainStride];
  __shared__ float red[kTrainWaves][64 + 64 + 16 + 1];
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // weight-gradient blocks wave, wave + 8, ...: 0-15 dW1, 16-31 dW2, 32-35 dW3
  constexpr int NB = (36 + kTrainWaves - 1) / kTrainWaves;
  double *rec = partial + (size_t)blockIdx.x * kMlpRecord;
  double *pW1 = rec, *pb1 = pW1 + 4096, *pW2 = pb1 + 64, *pb2 = pW2 + 4096, *pW3 = pb2 + 64,
         *pb3 = pW3 + 1024, *psse = pb3 + 16;
  constexpr bool LONG = RUN == 0;
  v4f held[LONG ? NB : 1];  // the chunks that the record does not have yet
#pragma unroll
  for (v4f &h : held) h = v4f{0, 0, 0, 0};
  v4f gb1[4], gb2[4], gb3 = {0, 0, 0, 0};
#pragma unroll
  for (int a = 0; a < 4; ++a) gb1[a] = gb2[a] = v4f{0, 0, 0, 0};
  float sse = 0.0f;
  InNorm nm;
  load_norm(mean, stdv, w.nin, g, nm);
  const long long nchunks = (n + kTrainNodes - 1) / kTrainNodes;
  int left = chunks;  // LONG: until the run's end
  bool first = true;  // the record is empty
  for (long long chunk = blockIdx.x; chunk < nchunks; chunk += gridDim.x) {
    const int col = 16 * wave + c;  // the node's column of the staging rows
    const long long node = chunk * kTrainNodes + col;
    const bool valid = node < n;
    Tile t;
    tile_inputs(nm, X, n, w.nin, node, g, t);
    tile_layers<true>(w, c, g, t);
    // output error (zero outside the valid nodes and outputs)
    v4f dy;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = 4 * g + i;
      float e = 0.0f;
      if (valid && o < w.nout) e = t.z3[i] - (T[node * w.nout + o] - w.out_mean[o]) / w.out_std[o];
      sse += e * e;
      dy[i] = scale * e;
    }
    gb3 += dy;
    const v4s dyb = pack4(dy);
    auto stage = [&](int first, int mb, const v4s &v) {  // four units of the lane's node
#pragma unroll
      for (int i = 0; i < 4; ++i) st[first + 16 * mb + 4 * g + i][col] = (uint16_t)v[i];
    };
    stage(320, 0, dyb);
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      stage(0, mb, t.x[mb]);
      stage(64, mb, t.h1[mb]);
      stage(128, mb, t.h2[mb]);
    }
    // dH2 = W3^T dY, dZ2 = dH2 gelu'(z2)
    v4s dz2b[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      v4f acc = mfma(ld4(w.W3Tb + (16 * mb + c) * 16 + 4 * g), dyb, v4f{0, 0, 0, 0});
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] *= t.d2[mb][i];
      dz2b[mb] = pack4(acc);
      gb2[mb] += acc;
      stage(256, mb, dz2b[mb]);
    }
    // dH1 = W2^T dZ2, dZ1 = dH1 gelu'(z1)
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      v4f acc = {0, 0, 0, 0};
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
        acc = mfma(ld4(w.W2Tb + (16 * mb + c) * 64 + 16 * kb + 4 * g), dz2b[kb], acc);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] *= t.d1[mb][i];
      gb1[mb] += acc;
      stage(192, mb, pack4(acc));
    }
    __syncthreads();
    // dW1 += dZ1^T X, dW2 += dZ2^T H1, dW3 += dY^T H2 (K = the chunk's nodes)
    const bool put = !LONG || --left == 0 || chunk + gridDim.x >= nchunks;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int b = wave + kTrainWaves * j;  // wave-uniform
      if (b < 36) {
        const int ra = b < 16 ? 192 + 16 * (b >> 2) : b < 32 ? 256 + 16 * ((b - 16) >> 2) : 320;
        const int rb = b < 16 ? 16 * (b & 3) : b < 32 ? 64 + 16 * (b & 3) : 128 + 16 * (b & 3);
        double sum[4] = {0.0, 0.0, 0.0, 0.0};
        v4f acc = LONG ? held[LONG ? j : 0] : v4f{0, 0, 0, 0};
#pragma unroll
        for (int kb = 0; kb < kTrainNodes / 16; ++kb) {
          acc = mfma(ld4(&st[ra + c][16 * kb + 4 * g]), ld4(&st[rb + c][16 * kb + 4 * g]), acc);
          if (kb == kTrainNodes / 16 - 1 ? put : !LONG && (kb + 1) % (LONG ? 1 : RUN) == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[i] += acc[i];
            acc = v4f{0, 0, 0, 0};
          }
        }
        if (LONG) held[LONG ? j : 0] = acc;
        if (put) {
          double *dst = b < 16 ? pW1 : b < 32 ? pW2 : pW3;
          const int mo = b < 32 ? (b & 15) >> 2 : 0, mi = b & 3;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            double &r = dst[(16 * mo + 4 * g + i) * 64 + 16 * mi + c];
            r = first ? sum[i] : r + sum[i];
          }
        }
      }
    }
    if (put) {
      left = chunks;
      first = false;
    }
    __syncthreads();  // the next chunk overwrites the staging rows
  }
  // bias gradients: sum over the 16 node columns of each lane group, then the waves
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        gb1[mb][i] += __shfl_xor(gb1[mb][i], m);
        gb2[mb][i] += __shfl_xor(gb2[mb][i], m);
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) gb3[i] += __shfl_xor(gb3[i], m);
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) sse += __shfl_xor(sse, m);
  if (c == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        red[wave][16 * mb + 4 * g + i] = gb1[mb][i];
        red[wave][64 + 16 * mb + 4 * g + i] = gb2[mb][i];
      }
      red[wave][128 + 4 * g + i] = gb3[i];
    }
    if (g == 0) red[wave][144] = sse;
  }
  __syncthreads();
  if (threadIdx.x < 145) {
    const int j = threadIdx.x;
    double s = 0.0;
    for (int v = 0; v < kTrainWaves; ++v) s += red[v][j];
    double *dst = j < 64 ? pb1 + j : j < 128 ? pb2 + j - 64 : j < 144 ? pb3 + j - 128 : psse;
    *dst = s;
  }
}

// Record position -> canonical position (parameters, then the sum of squared
// errors at nparams), or -1 for padding.
__device__ __forceinline__ int canonical(int j, int nin, int nout) {
  const int ob1 = 64 * nin, oW2 = ob1 + 64, ob2 = oW2 + 4096, oW3 = ob2 + 64,
            ob3 = oW3 + 64 * nout, osse = ob3 + nout;
  if (j < 4096) return j % 64 < nin ? (j / 64) * nin + j % 64 : -1;
  if (j < 4160) return ob1 + (j - 4096);
  if (j < 8256) return oW2 + (j - 4160);
  if (j < 8320) return ob2 + (j - 8256);
  if (j < 9344) return (j - 8320) / 64 < nout ? oW3 + (j - 8320) : -1;
  if (j < 9360) return j - 9344 < nout ? ob3 + (j - 9344) : -1;
  return osse;
}

// A parameter's copies in the operand arrays (BF16 weights, zero padded by
// k_mlp_pack, W2 and W3 also transposed; padded FP32 biases); j is its record
// position.
__device__ __forceinline__ void put_operand(int j, float v, const MlpDev &w) {
  uint16_t *W1b = const_cast<uint16_t *>(w.W1b), *W2b = const_cast<uint16_t *>(w.W2b),
           *W3b = const_cast<uint16_t *>(w.W3b), *W2Tb = const_cast<uint16_t *>(w.W2Tb),
           *W3Tb = const_cast<uint16_t *>(w.W3Tb);
  const uint16_t h = (uint16_t)bf16_bits(v);
  if (j < 4096) {
    W1b[j] = h;
  } else if (j < 4160) {
    const_cast<float *>(w.b1)[j - 4096] = v;
  } else if (j < 8256) {
    const int i = j - 4160;
    W2b[i] = h;
    W2Tb[(i % 64) * 64 + i / 64] = h;
  } else if (j < 8320) {
    const_cast<float *>(w.b2)[j - 8256] = v;
  } else if (j < 9344) {
    const int i = j - 8320;
    W3b[i] = h;
    W3Tb[(i % 64) * 16 + i / 64] = h;
  } else {
    const_cast<float *>(w.b3)[j - 9344] = v;
  }
}

// Adam's constants of one step (Kingma & Ba 2015); bias corrections c1, c2.
struct AdamStep {
  float *theta, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};

// Sum the workgroups' records in FP64 (fixed order) into grad (canonical
// layout, then the sum of squared errors); with ADAM also take the step on
// the FP32 master parameters and renew their operand copies.  32 record
// positions per workgroup, eight threads each: a thread that walks all the
// records of its position alone takes 126 us for 512 of them on 37
// workgroups, and Adam and the packing were two more launches (11 us); here 7.
template <bool ADAM>
__global__ void __launch_bounds__(256)
    k_mlp_reduce(const double *__restrict__ partial, int nrec, MlpDev w, float *__restrict__ grad,
                 AdamStep ad) {
  __shared__ double part[8][32];
  const int jj = threadIdx.x & 31, sl = threadIdx.x >> 5;
  const int j = blockIdx.x * 32 + jj;
  double s = 0.0;
  if (j < kMlpRecord) {
#pragma unroll 8
    for (int r = sl; r < nrec; r += 8) s += partial[(size_t)r * kMlpRecord + j];
  }
  part[sl][jj] = s;
  __syncthreads();
  if (sl != 0 || j >= kMlpRecord) return;
  for (int i = 1; i < 8; ++i) s += part[i][jj];
  const int dst = canonical(j, w.nin, w.nout);
  if (dst < 0) return;
  const float gj = (float)s;
  grad[dst] = gj;
  if (ADAM && j < kMlpRecord - 1) {
    const float mj = ad.b1 * ad.m[dst] + (1.0f - ad.b1) * gj;
    const float vj = ad.b2 * ad.v[dst] + (1.0f - ad.b2) * gj * gj;
    ad.m[dst] = mj;
    ad.v[dst] = vj;
    const float th = ad.theta[dst] - ad.lr * (mj / ad.c1) / (sqrtf(vj / ad.c2) + ad.eps);
    ad.theta[dst] = th;
    put_operand(j, th, w);
  }
}

// Canonical FP32 parameters -> BF16 operand arrays (zero padded) and
// padded FP32 biases: W1b [64][64], W2b [64][64], W3b [16][64],
// W2Tb [64][64] (transposed), W3Tb [64][16] (transposed).
__global__ void k_mlp_pack(const float *__restrict__ theta, int nin, int nout,
                           uint16_t *__restrict__ W1b, uint16_t *__restrict__ W2b,
                           uint16_t *__restrict__ W3b, uint16_t *__restrict__ W2Tb,
                           uint16_t *__restrict__ W3Tb, float *__restrict__ b1,
                           float *__restrict__ b2, float *__restrict__ b3) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const float *W1 = theta, *B1 = W1 + 64 * nin, *W2 = B1 + 64, *B2 = W2 + 4096, *W3 = B2 + 64,
              *B3 = W3 + 64 * nout;
  if (j < 4096) {
    const int r = j / 64, k = j % 64;
    W1b[j] = (uint16_t)bf16_bits(k < nin ? W1[r * nin + k] : 0.0f);
    W2b[j] = (uint16_t)bf16_bits(W2[j]);
    W2Tb[j] = (uint16_t)bf16_bits(W2[k * 64 + r]);  // W2Tb[r][k] = W2[k][r]
  }
  if (j < 1024) {
    const int o = j / 64, h = j % 64;
    W3b[j] = (uint16_t)bf16_bits(o < nout ? W3[o * 64 + h] : 0.0f);
    const int hh = j / 16, oo = j % 16;
    W3Tb[j] = (uint16_t)bf16_bits(oo < nout ? W3[oo * 64 + hh] : 0.0f);
  }
  if (j < 64) {
    b1[j] = B1[j];
    b2[j] = B2[j];
  }
  if (j < 16) b3[j] = j < nout ? B3[j] : 0.0f;
}

// ---------------------------------------------------------------------------
// Lattice side (FP64).

// Features of every node from the observables obs[10][N]: the 3x3 periodic
// neighbourhood of rho, Ux, Uy, Cxx, Cxy, Cyy, feature 6 s + f for stencil
// position s = 3 (dy + 1) + (dx + 1).  Raw values to X [N][54] (if X) and
// standardised BF16 rows to Xb [N][64] (if Xb).
__global__ void k_features(const double *__restrict__ obs, int nx, int ny,
                           const float *__restrict__ mean, const float *__restrict__ stdv,
                           float *__restrict__ X, uint16_t *__restrict__ Xb) {
  const long long N = (long long)nx * ny;
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= N) return;
  const int y = (int)(r / nx), x = (int)(r - (long long)y * nx);
  const int fields[6] = {0, 1, 2, 4, 5, 6};
#pragma unroll
  for (int s = 0; s < 9; ++s) {
    const int yy = (y + s / 3 - 1 + ny) % ny, xx = (x + s % 3 - 1 + nx) % nx;
    const long long rr = (long long)yy * nx + xx;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      const float v = (float)obs[(size_t)fields[f] * N + rr];
      const int k = 6 * s + f;
      if (X) X[r * 54 + k] = v;
      if (Xb) Xb[r * 64 + k] = (uint16_t)bf16_bits((v - mean[k]) / stdv[k]);
    }
  }
  if (Xb)
    for (int k = 54; k < 64; ++k) Xb[r * 64 + k] = 0;
}

// Targets [N][5]: (rho U, tau) of obs_ref minus those of obs.
__global__ void k_targets(const double *__restrict__ ref, const double *__restrict__ obs,
                          long long N, float *__restrict__ T) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= N) return;
  auto ms = [&](const double *o, int j) -> double {
    switch (j) {
      case 0: return o[r] * o[N + r];
      case 1: return o[r] * o[2 * N + r];
      default: return o[(size_t)(5 + j) * N + r];
    }
  };
#pragma unroll
  for (int j = 0; j < 5; ++j) T[r * 5 + j] = (float)(ms(ref, j) - ms(obs, j));
}

// Momentum source F [2][N] = dJ + div_h(dtau) (central differences) from a
// correction corr [N][5] (dJx, dJy, dtau_xx, dtau_xy, dtau_yy).
__global__ void k_source(const float *__restrict__ corr, int nx, int ny,
                         double *__restrict__ F) {
  const long long N = (long long)nx * ny;
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= N) return;
  const int y = (int)(r / nx), x = (int)(r - (long long)y * nx);
  const long long e = (long long)y * nx + (x + 1) % nx, wv = (long long)y * nx + (x - 1 + nx) % nx;
  const long long nn = (long long)((y + 1) % ny) * nx + x, s = (long long)((y - 1 + ny) % ny) * nx + x;
  auto cc = [&](long long i, int j) -> double { return (double)corr[i * 5 + j]; };
  F[r] = cc(r, 0) + 0.5 * (cc(e, 2) - cc(wv, 2)) + 0.5 * (cc(nn, 3) - cc(s, 3));
  F[N + r] = cc(r, 1) + 0.5 * (cc(e, 3) - cc(wv, 3)) + 0.5 * (cc(nn, 4) - cc(s, 4));
}

// Per-workgroup sums of both source components, partial[blk][2] (fixed
// order: the removal of the mean below is deterministic).
__global__ void k_source_sums(const double *__restrict__ F, long long N,
                              double *__restrict__ partial) {
  __shared__ double sx[256], sy[256];
  double a = 0.0, b = 0.0;
  for (long long r = (long long)blockIdx.x * 256 + threadIdx.x; r < N;
       r += (long long)gridDim.x * 256) {
    a += F[r];
    b += F[N + r];
  }
  sx[threadIdx.x] = a;
  sy[threadIdx.x] = b;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      sx[threadIdx.x] += sx[threadIdx.x + s];
      sy[threadIdx.x] += sy[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = sx[0];
    partial[2 * blockIdx.x + 1] = sy[0];
  }
}

// F -= sum / N per component.
__global__ void k_source_center(double *__restrict__ F, long long N,
                                const double *__restrict__ sums) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= N) return;
  const double mx = sums[0] / (double)N, my = sums[1] / (double)N;
  F[r] -= mx;
  F[N + r] -= my;
}

// Largest |F| / rho over the lattice, per workgroup into partial[] (the
// velocity change a source makes in one step).
__global__ void k_source_drift(const double *__restrict__ F, const double *__restrict__ FLD,
                               long long N, double *__restrict__ partial) {
  __shared__ double sh[256];
  double mx = 0.0;
  for (long long r = (long long)blockIdx.x * 256 + threadIdx.x; r < N;
       r += (long long)gridDim.x * 256) {
    const double rho = FLD[(size_t)F_RHOS * N + r] + FLD[(size_t)F_RHOP * N + r];
    const double f = sqrt(F[r] * F[r] + F[N + r] * F[N + r]) / rho;
    mx = (f > mx || !(f == f)) ? f : mx;  // NaN wins
  }
  sh[threadIdx.x] = mx;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      const double o = sh[threadIdx.x + s];
      if (o > sh[threadIdx.x] || !(o == o)) sh[threadIdx.x] = o;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

// Full-weighting restriction by an even factor m of planes of a fine
// lattice (nxf x nyf) onto a coarse one: coarse (X, Y) averages fine
// (m X + i, m Y + j), |i|, |j| <= m/2, weights 1/2 on the window's edges.
// This form, one thread per coarse value, takes any factor.
template <typename T>
__global__ void k_restrict(int planes, int nxf, int nyf, int m, const T *__restrict__ src,
                           double *__restrict__ dst) {
  const int nxc = nxf / m, nyc = nyf / m;
  const long long Nc = (long long)nxc * nyc, Nf = (long long)nxf * nyf;
  const long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= Nc * planes) return;
  const int pl = (int)(j / Nc);
  const long long rc = j - (long long)pl * Nc;
  const int Y = (int)(rc / nxc), X = (int)(rc - (long long)Y * nxc);
  const T *P = src + (size_t)pl * Nf;
  const int h = m / 2;
  double acc = 0.0;
  for (int dj = -h; dj <= h; ++dj) {
    const double wy = (dj == -h || dj == h) ? 0.5 : 1.0;
    const int y = (m * Y + dj + nyf) % nyf;
    double row = 0.0;
    for (int di = -h; di <= h; ++di) {
      const double wx = (di == -h || di == h) ? 0.5 : 1.0;
      const int x = (m * X + di + nxf) % nxf;
      row += wx * (double)P[(long long)y * nxf + x];
    }
    acc += wy * row;
  }
  dst[(size_t)pl * Nc + rc] = acc / ((double)m * m);
}

// The same for m = 2 and 4, same sums in the same order.  Bound by the one
// read of the fine planes, so every fine row is read once, in order: lane X
// of a wave reads its M values of a row (and the M / 2 before them, its left
// neighbour's, from the cache), and the wave walks kRestrictRows coarse rows
// down, keeping the row sum that two coarse rows share.  The thread-per-value
// form reads each fine row 1.25 times at stride M (1024^2 to 256^2, 1300
// planes, with the refresh: 3.7 ms a call against 2.6; 5.0 TB/s).
constexpr int kRestrictRows = 8;
template <int M>
__global__ void __launch_bounds__(256)
    k_restrict_rows(int planes, int nxf, int nyf, const double *__restrict__ src,
                    double *__restrict__ dst) {
  constexpr int h = M / 2;
  typedef double vm __attribute__((ext_vector_type(M)));
  typedef double vh __attribute__((ext_vector_type(h)));
  const int nxc = nxf / M, nyc = nyf / M;
  const int X = blockIdx.x * 64 + (threadIdx.x & 63);
  const int pl = blockIdx.z * 4 + (threadIdx.x >> 6);
  if (pl >= planes || X >= nxc) return;
  const double *P = src + (size_t)pl * nxf * nyf;
  double *D = dst + (size_t)pl * nxc * nyc;
  const int x0 = M * X, xl = X == 0 ? nxf - h : x0 - h;
  // sum over the window's columns of fine row y
  auto row = [&](int y) {
    const vm v = *reinterpret_cast<const vm *>(P + (size_t)y * nxf + x0);
    const vh l = *reinterpret_cast<const vh *>(P + (size_t)y * nxf + xl);
    double lv[h], vv[M];
    __builtin_memcpy(lv, &l, sizeof lv);
    __builtin_memcpy(vv, &v, sizeof vv);
    double s = 0.5 * lv[0];
#pragma unroll
    for (int i = 1; i < h; ++i) s += lv[i];
#pragma unroll
    for (int i = 0; i < h; ++i) s += vv[i];
    return s + 0.5 * vv[h];
  };
  const int Y0 = blockIdx.y * kRestrictRows;
  const int Y1 = Y0 + kRestrictRows < nyc ? Y0 + kRestrictRows : nyc;
  double edge = row(Y0 == 0 ? nyf - h : M * Y0 - h);
  for (int Y = Y0; Y < Y1; ++Y) {
    double r[M];
#pragma unroll
    for (int j = 0; j < M; ++j) r[j] = row(M * Y - h + 1 + j < 0 ? M * Y - h + 1 + j + nyf
                                                                  : M * Y - h + 1 + j);
    double acc = 0.5 * edge;
#pragma unroll
    for (int j = 0; j < M - 1; ++j) acc += r[j];
    edge = r[M - 1];
    acc += 0.5 * edge;
    D[(size_t)Y * nxc + X] = acc / (double)(M * M);
  }
}

// ---------------------------------------------------------------------------
// The attached correction of a coarse step, fused.

// Feature k of node (x, y) from the observables, as k_features computes it:
// field f = k % 6 of (rho, Ux, Uy, Cxx, Cxy, Cyy) at stencil position
// s = k / 6 = 3 (dy + 1) + (dx + 1), periodic.
__device__ __forceinline__ float stencil_feature(const double *__restrict__ obs, int nx, int ny,
                                                 int x, int y, int k) {
  const int s = k / 6, f = k - 6 * s;
  const int fld = f < 3 ? f : f + 1;
  const int yy = (y + s / 3 - 1 + ny) % ny, xx = (x + s % 3 - 1 + nx) % nx;
  return (float)obs[(size_t)fld * nx * ny + (size_t)yy * nx + xx];
}

// One wave per 16-node tile: features, network, correction in physical
// units, and the wave's sums of the two momentum corrections.
__global__ void __launch_bounds__(256) k_correct(MlpDev w, const double *__restrict__ obs, int nx,
                                                 int ny, const float *__restrict__ mean,
                                                 const float *__restrict__ stdv,
                                                 float *__restrict__ corr,
                                                 double *__restrict__ partial,
                                                 const int *__restrict__ gate) {
  if (*gate) return;  // uniform: the drift gate stopped an earlier step
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const long long N = (long long)nx * ny;
  const long long wid = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const long long n0 = wid * 16, node = n0 + c;
  const bool valid = node < N;
  double jx = 0.0, jy = 0.0;
  if (n0 < N) {  // whole wave
    Tile t;
    const int y = valid ? (int)(node / nx) : 0, x = valid ? (int)(node - (long long)y * nx) : 0;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      v4s v = {0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = 16 * kb + 4 * g + i;
        if (valid && k < w.nin)
          v[i] = bf16_bits((stencil_feature(obs, nx, ny, x, y, k) - mean[k]) / stdv[k]);
      }
      t.x[kb] = v;
    }
    tile_layers<false>(w, c, g, t);
    if (valid)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int o = 4 * g + i;
        if (o < w.nout) {
          const float v = t.z3[i] * w.out_std[o] + w.out_mean[o];
          corr[node * w.nout + o] = v;
          if (o == 0) jx = (double)v;
          if (o == 1) jy = (double)v;
        }
      }
  }
  jx = wave_sum(jx);
  jy = wave_sum(jy);
  if (lane == 0 && n0 < N) {  // one record per wave of correct_waves(N)
    partial[2 * wid] = jx;
    partial[2 * wid + 1] = jy;
  }
}

// F = (dJ - <dJ>) + div_h(dtau) and the drift gate (grid-stride; every
// workgroup forms the lattice mean from the per-wave sums in one fixed
// order).
__global__ void __launch_bounds__(256) k_source_gate(const float *__restrict__ corr, int nx,
                                                     int ny, const double *__restrict__ partial,
                                                     long long nparts,
                                                     const double *__restrict__ FLD, double bound,
                                                     int tag, double *__restrict__ F,
                                                     int *__restrict__ gate,
                                                     unsigned long long *__restrict__ drift) {
  __shared__ double sh[16];
  if (*gate) return;  // uniform
  const long long N = (long long)nx * ny;
  double sx = 0.0, sy = 0.0;
  // every workgroup sums all records: eight loads in flight, added in order
  // (65536 nodes, 4096 records: the kernel 10.6 us one by one, 8.0 so)
  long long i = threadIdx.x;
  for (; i + 7 * 256 < nparts; i += 8 * 256) {
    double a[8], b[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      a[j] = partial[2 * (i + 256 * j)];
      b[j] = partial[2 * (i + 256 * j) + 1];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      sx += a[j];
      sy += b[j];
    }
  }
  for (; i < nparts; i += 256) {
    sx += partial[2 * i];
    sy += partial[2 * i + 1];
  }
  const double mx = block_sum(sx, sh) / (double)N, my = block_sum(sy, sh) / (double)N;
  double dmax = 0.0;
  for (long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x; r < N;
       r += (long long)gridDim.x * blockDim.x) {
    const int y = (int)(r / nx), x = (int)(r - (long long)y * nx);
    const long long e = (long long)y * nx + (x + 1) % nx, wv = (long long)y * nx + (x - 1 + nx) % nx;
    const long long nn = (long long)((y + 1) % ny) * nx + x, s = (long long)((y - 1 + ny) % ny) * nx + x;
    auto cc = [&](long long i, int j) -> double { return (double)corr[i * 5 + j]; };
    const double fx = cc(r, 0) - mx + 0.5 * (cc(e, 2) - cc(wv, 2)) + 0.5 * (cc(nn, 3) - cc(s, 3));
    const double fy = cc(r, 1) - my + 0.5 * (cc(e, 3) - cc(wv, 3)) + 0.5 * (cc(nn, 4) - cc(s, 4));
    F[r] = fx;
    F[N + r] = fy;
    const double rho = FLD[(size_t)F_RHOS * N + r] + FLD[(size_t)F_RHOP * N + r];
    const double d = sqrt(fx * fx + fy * fy) / rho;
    dmax = (d > dmax || !(d == d)) ? d : dmax;  // NaN wins
  }
  // a NaN anywhere in the workgroup makes its maximum infinite
  const double bad = block_sum(dmax == dmax ? 0.0 : 1.0, sh);
  dmax = bad > 0.0 ? INFINITY : block_max(dmax, sh);
  if (threadIdx.x == 0) {
    atomicMax(drift, (unsigned long long)__double_as_longlong(dmax));
    if (!(dmax <= bound)) atomicCAS(gate, 0, tag);
  }
}

// ---------------------------------------------------------------------------
// Launchers

hipError_t launch_mlp_forward(const MlpDev &w, const float *mean, const float *stdv,
                              const float *X, long long n, float *Y, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const long long tiles = (n + 15) / 16;
  hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, s, w, mean,
                     stdv, X, n, Y);
  return hipGetLastError();
}

int mlp_records(long long n) {
  const long long chunks = (n + kTrainNodes - 1) / kTrainNodes;
  return (int)std::min<long long>(chunks, kMlpRecs);
}

hipError_t launch_mlp_train(const MlpDev &w, const float *mean, const float *stdv, const float *X,
                            const float *T, long long n, double *partial, hipStream_t s) {
  const float scale = 2.0f / (float)((double)n * w.nout);
  // a run's tiles: at most a 512th of all (rounded up)
  const long long most = ((n + 15) / 16 + 511) / 512;
  auto kernel = most >= 2 * kTrainWaves ? k_mlp_train<0>
                : most >= kTrainWaves   ? k_mlp_train<kTrainWaves>
                                        : k_mlp_train<1>;
  hipLaunchKernelGGL(kernel, dim3(mlp_records(n)), dim3(64 * kTrainWaves), 0, s, w, mean, stdv, X,
                     T, n, scale, (int)std::min(most / kTrainWaves, 1LL << 30), partial);
  return hipGetLastError();
}

hipError_t launch_mlp_reduce(const double *partial, long long n, const MlpDev &w, float *grad,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_reduce<false>, dim3((kMlpRecord + 31) / 32), dim3(256), 0, s, partial,
                     mlp_records(n), w, grad, AdamStep{});
  return hipGetLastError();
}

hipError_t launch_mlp_update(const double *partial, long long n, const MlpDev &w, float *grad,
                             float *theta, float *m, float *v, float lr, int t, hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float c1 = (float)(1.0 - std::pow(0.9, t)), c2 = (float)(1.0 - std::pow(0.999, t));
  const AdamStep ad{theta, m, v, lr, b1, b2, eps, c1, c2};
  hipLaunchKernelGGL(k_mlp_reduce<true>, dim3((kMlpRecord + 31) / 32), dim3(256), 0, s, partial,
                     mlp_records(n), w, grad, ad);
  return hipGetLastError();
}

hipError_t launch_mlp_pack(const float *theta, int nin, int nout, const MlpDev &w,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_pack, dim3(16), dim3(256), 0, s, theta, nin, nout,
                     const_cast<uint16_t *>(w.W1b), const_cast<uint16_t *>(w.W2b),
                     const_cast<uint16_t *>(w.W3b), const_cast<uint16_t *>(w.W2Tb),
                     const_cast<uint16_t *>(w.W3Tb), const_cast<float *>(w.b1),
                     const_cast<float *>(w.b2), const_cast<float *>(w.b3));
  return hipGetLastError();
}

hipError_t launch_features(const double *obs, int nx, int ny, const float *mean,
                           const float *stdv, float *X, uint16_t *Xb, hipStream_t s) {
  const long long N = (long long)nx * ny;
  hipLaunchKernelGGL(k_features, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, obs, nx,
                     ny, mean, stdv, X, Xb);
  return hipGetLastError();
}

hipError_t launch_targets(const double *ref, const double *obs, long long N, float *T,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_targets, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, ref, obs, N,
                     T);
  return hipGetLastError();
}

hipError_t launch_source(const float *corr, int nx, int ny, double *F, hipStream_t s) {
  const long long N = (long long)nx * ny;
  hipLaunchKernelGGL(k_source, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, corr, nx, ny,
                     F);
  return hipGetLastError();
}

hipError_t launch_source_center(double *F, long long N, double *scratch, hipStream_t s) {
  const long long nb = std::min<long long>(1024, (N + 255) / 256);
  hipLaunchKernelGGL(k_source_sums, dim3((unsigned)nb), dim3(256), 0, s, F, N, scratch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_sum(scratch, (int)nb, 2, scratch + 2048, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_source_center, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, F, N,
                     scratch + 2048);
  return hipGetLastError();
}

hipError_t launch_source_drift(const double *F, const double *FLD, long long N, double *partial,
                               int *nblocks, hipStream_t s) {
  const long long nb = std::min<long long>(1024, (N + 255) / 256);
  *nblocks = (int)nb;
  hipLaunchKernelGGL(k_source_drift, dim3((unsigned)nb), dim3(256), 0, s, F, FLD, N, partial);
  return hipGetLastError();
}

long long correct_waves(long long N) { return (N + 15) / 16; }

hipError_t launch_correct(const MlpDev &w, const double *obs, int nx, int ny, const float *mean,
                          const float *stdv, float *corr, double *partial, const int *gate,
                          hipStream_t s) {
  const long long waves = correct_waves((long long)nx * ny);
  hipLaunchKernelGGL(k_correct, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, w, obs, nx,
                     ny, mean, stdv, corr, partial, gate);
  return hipGetLastError();
}

hipError_t launch_source_gate(const float *corr, int nx, int ny, const double *partial,
                              long long nparts, const double *FLD, double bound, int tag,
                              double *F, int *gate, unsigned long long *drift, hipStream_t s) {
  const long long N = (long long)nx * ny;
  long long nb = (N + 255) / 256;
  if (nb > 128) nb = 128;
  hipLaunchKernelGGL(k_source_gate, dim3((unsigned)nb), dim3(256), 0, s, corr, nx, ny, partial,
                     nparts, FLD, bound, tag, F, gate, drift);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_restrict(int planes, int nxf, int nyf, int m, const T *src, double *dst,
                           hipStream_t s) {
  const long long n = (long long)(nxf / m) * (nyf / m) * planes;
  const int nxc = nxf / m, nyc = nyf / m;
  // rows of M doubles start 16-byte aligned if src does: nxf is a multiple of m
  const bool rows = std::is_same<T, double>::value && (m == 2 || m == 4) &&
                    reinterpret_cast<uintptr_t>(src) % (8 * m) == 0 && planes <= 4 * 65535;
  if (rows) {
    const dim3 grid((nxc + 63) / 64, (nyc + kRestrictRows - 1) / kRestrictRows, (planes + 3) / 4);
    if (grid.y <= 65535) {
      const double *p = reinterpret_cast<const double *>(src);
      if (m == 4)
        hipLaunchKernelGGL(k_restrict_rows<4>, grid, dim3(256), 0, s, planes, nxf, nyf, p, dst);
      else
        hipLaunchKernelGGL(k_restrict_rows<2>, grid, dim3(256), 0, s, planes, nxf, nyf, p, dst);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL(k_restrict<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, planes,
                     nxf, nyf, m, src, dst);
  return hipGetLastError();
}
template hipError_t launch_restrict<double>(int, int, int, int, const double *, double *,
                                            hipStream_t);

}  // namespace tplk
