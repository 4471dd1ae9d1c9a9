// fr_mlp.hip -- the per-element network of the learned eddy-viscosity closure on gfx950.
//
// Forward and backward passes run four wavefronts per 16 samples on the matrix cores
// (v_mfma_f32_16x16x16_bf16, float32 accumulation), each wave a 16-unit block of every layer's
// output. With that instruction a wave holds the 16x16 result tile D[m][n] as lane (g = lane/16,
// c = lane%16) -> rows 4g..4g+3 of column c, which is the lane layout of its B operand (rows k =
// 4g..4g+3 of column c): a layer's output goes to the next through LDS as [sample][unit], four
// units per 16-byte access.
//
// Weights are the bfloat16 roundings of float32 masters. An activation x enters a product as
// hi + lo, hi = bf16(x), lo = bf16(x - hi) (two MFMAs), which represents it to 2^-17 relative,
// so the products see the weights exactly and the activations nearly exactly.
//
// Training: after the backward pass each wave adds the 16 samples' outer products to its rows of
// the weight gradients on the matrix cores (dW = delta^T h with both operands split: hi*hi + hi*lo +
// lo*hi), which it keeps in registers over all of the block's samples and writes as one partial sum
// per block. The Adam kernel adds the partials in a fixed
// order and updates the masters and their bf16 copies. There are no atomics: every result is
// deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "fr.h"
#include "fr_internal.h"

using namespace frk;

namespace {

constexpr int H = 64;         // hidden units per layer
constexpr int kMaxIn = 128;   // inputs (padded to a multiple of 16)
constexpr int kChunk = 16;    // samples a block takes at a time
constexpr int kMaxPart = 256; // blocks of the training pass, each with a partial sum of the gradient

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short bf16_bits(float x) {
  unsigned u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest, ties to even (finite inputs)
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_val(unsigned short b) { return __uint_as_float((unsigned)b << 16); }

__device__ __forceinline__ v4f mfma(v4s a, v4s b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float softplus(float z) { return z > 20.f ? z : log1pf(expf(z)); }
__device__ __forceinline__ float logistic(float z) { return 1.f / (1.f + expf(-z)); }

// Device state of one network.
struct Net {
  int F, FP;                 // inputs; padded to a multiple of 16
  int64_t np;                // parameters
  int64_t oW1, ob1, oW2, ob2, ow3, ob3;
  float *theta = nullptr;    // float32 masters [np]
  float *am = nullptr;       // Adam first moments [np]
  float *av = nullptr;       // Adam second moments [np]
  unsigned short *W1b = nullptr;   // [H][FP] bf16, zero padded
  unsigned short *W2b = nullptr;   // [H][H]
  unsigned short *W2Tb = nullptr;  // [H][H] transposed
  float *w3r = nullptr;      // [H] bf16-rounded w3 as float
  float *mean = nullptr;     // [FP] (0 beyond F)
  float *istd = nullptr;     // [FP] 1/std (0 beyond F)
  float *part = nullptr;     // training scratch: [blocks][np + 1] partial gradients and losses
  int64_t part_cap = 0;
  float *grad = nullptr;     // [np]
  float *dloss = nullptr;    // [1]
  int step = 0;
};

struct NetArgs {
  int F, FP;
  const unsigned short *W1b, *W2b, *W2Tb;
  const float *b1, *b2, *w3r, *b3, *mean, *istd;
  // offsets of the parameters in a partial gradient (training)
  int64_t np, oW1, ob1, oW2, ob2, ow3, ob3;
};

// ------------------------------------------------------------------------------------------
// Forward pass of 16 samples per block, a quarter of each layer's units per wave; TRAIN: also the
// loss, the back-propagated deltas and this block's share of the gradient.
//
// A pass over a few thousand samples is bound by the instructions one wave issues in turn (splits,
// tanh): with a wave for all 64 units of 16 samples, 4096 samples kept one SIMD in four busy.
// Each wave keeps its rows of the weights in registers. 4096 samples of 68 inputs (us): evaluation
// 10.6 -> 4.9; training pass 20.4 and a separate gradient kernel 67.5 -> 12.5 for both.
// ------------------------------------------------------------------------------------------
// A value in the products: its hi and lo halves in one word.
__device__ __forceinline__ unsigned pack_hl(float x) {
  const unsigned short h = bf16_bits(x);
  return (unsigned)h | ((unsigned)bf16_bits(x - bf16_val(h)) << 16);
}
__device__ __forceinline__ void unpack_hl(const unsigned u[4], v4s &hi, v4s &lo) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    hi[i] = (short)(u[i] & 0xffffu);
    lo[i] = (short)(u[i] >> 16);
  }
}

// Sum over the 16 lanes of a row, on every one of them (rotations within the row).
template <int R>
__device__ __forceinline__ float row_ror(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 | R, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_sum(float x) {
  x += row_ror<8>(x);
  x += row_ror<4>(x);
  x += row_ror<2>(x);
  return x + row_ror<1>(x);
}

// Row strides in LDS: 16-byte aligned, and lanes of different rows on different banks.
constexpr int kRowH = H + 4;

// Four consecutive entries of a packed row (a B operand's four rows of one sample).
__device__ __forceinline__ void operand(const unsigned *row, v4s &hi, v4s &lo) {
  const uint4 w = *(const uint4 *)row;
  const unsigned u[4] = {w.x, w.y, w.z, w.w};
  unpack_hl(u, hi, lo);
}
// One unit's entries of samples 4 g .. 4 g + 3: an operand whose K runs over the samples.
template <int ROW>
__device__ __forceinline__ void operand_samples(const unsigned *tab, int g, int unit, v4s &hi, v4s &lo) {
  unsigned u[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) u[i] = tab[(4 * g + i) * ROW + unit];
  unpack_hl(u, hi, lo);
}
__device__ __forceinline__ void put4(unsigned *row, const float x[4]) {
  *(uint4 *)row = make_uint4(pack_hl(x[0]), pack_hl(x[1]), pack_hl(x[2]), pack_hl(x[3]));
}

template <int KT, bool TRAIN>
__global__ __launch_bounds__(256) void k_mlp(NetArgs a, const float *__restrict__ X, int64_t n, int64_t ldx,
                                             float *__restrict__ y, double *__restrict__ nu, double nu_scale,
                                             const float *__restrict__ tgt, float inv_n, float *__restrict__ part) {
  constexpr int FP = 16 * KT, kRowX = FP + 4;
  // the samples' inputs, activations and deltas, [sample][unit] (packed; sZ: h2 as floats)
  __shared__ alignas(16) unsigned sX[kChunk * kRowX];
  __shared__ alignas(16) unsigned sH1[kChunk * kRowH];
  __shared__ alignas(16) float sZ[kChunk * kRowH];
  __shared__ alignas(16) unsigned sD2[TRAIN ? kChunk * kRowH : 4];
  __shared__ alignas(16) unsigned sD1[TRAIN ? kChunk * kRowH : 4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int u0 = 16 * wave + 4 * g;  // this lane's four units of its wave's block
  // this wave's rows of the weights (A operands), biases and output weights
  v4s w1[KT], w2[4], w2t[4];
#pragma unroll
  for (int kk = 0; kk < KT; ++kk) w1[kk] = *(const v4s *)&a.W1b[(16 * wave + c) * FP + 16 * kk + 4 * g];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    w2[kk] = *(const v4s *)&a.W2b[(16 * wave + c) * H + 16 * kk + 4 * g];
    if (TRAIN) w2t[kk] = *(const v4s *)&a.W2Tb[(16 * wave + c) * H + 16 * kk + 4 * g];
  }
  const float4 b1 = *(const float4 *)&a.b1[u0], b2 = *(const float4 *)&a.b2[u0];
  float w3[4][4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const float4 q = *(const float4 *)&a.w3r[16 * t + 4 * g];
    w3[t][0] = q.x;
    w3[t][1] = q.y;
    w3[t][2] = q.z;
    w3[t][3] = q.w;
  }
  const float4 w3o = *(const float4 *)&a.w3r[u0];
  const float w3u[4] = {w3o.x, w3o.y, w3o.z, w3o.w};
  const float b3 = a.b3[0];
  // rows of whole 16-byte groups are read with 16-byte loads
  const bool vec = (ldx & 3) == 0 && ((uintptr_t)X & 15) == 0;
  v4f gW1[TRAIN ? KT : 1], gW2[TRAIN ? 4 : 1];  // gradient tiles: row block `wave`, every column block
  float vd1[4] = {0.f, 0.f, 0.f, 0.f}, vd2[4] = {0.f, 0.f, 0.f, 0.f}, vw3[4] = {0.f, 0.f, 0.f, 0.f};
  float vz = 0.f, vl = 0.f;
  if (TRAIN) {
#pragma unroll
    for (int t = 0; t < KT; ++t) gW1[t] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) gW2[t] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  for (int64_t chunk = blockIdx.x; chunk * kChunk < n; chunk += gridDim.x) {
    const int64_t s = chunk * kChunk + c;  // this lane's sample
    const bool ok = s < n;
    const float target = TRAIN && ok ? tgt[s] : 0.f;
    // standardised inputs, K-steps shared out over the waves: rows k = 16 kk + 4 g + i
#pragma unroll
    for (int kk = wave; kk < KT; kk += 4) {
      const int k0 = 16 * kk + 4 * g;
      float x[4] = {0.f, 0.f, 0.f, 0.f};
      if (vec && ok && k0 + 3 < a.F) {
        const float4 q = *(const float4 *)&X[s * ldx + k0];
        x[0] = q.x;
        x[1] = q.y;
        x[2] = q.z;
        x[3] = q.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (ok && k0 + i < a.F) x[i] = X[s * ldx + k0 + i];
      }
      const float4 mu = *(const float4 *)&a.mean[k0], is = *(const float4 *)&a.istd[k0];
      const float m4[4] = {mu.x, mu.y, mu.z, mu.w}, i4[4] = {is.x, is.y, is.z, is.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = (ok && k0 + i < a.F) ? (x[i] - m4[i]) * i4[i] : 0.f;
      put4(&sX[c * kRowX + k0], x);
    }
    __syncthreads();
    // layer 1
    float h1[4], h2[4];
    {
      v4f acc = {b1.x, b1.y, b1.z, b1.w};
#pragma unroll
      for (int kk = 0; kk < KT; ++kk) {
        v4s bh, bl;
        operand(&sX[c * kRowX + 16 * kk + 4 * g], bh, bl);
        acc = mfma(w1[kk], bh, acc);
        acc = mfma(w1[kk], bl, acc);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) h1[i] = tanhf(acc[i]);
    }
    put4(&sH1[c * kRowH + u0], h1);
    __syncthreads();
    // layer 2
    {
      v4f acc = {b2.x, b2.y, b2.z, b2.w};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        v4s bh, bl;
        operand(&sH1[c * kRowH + 16 * kk + 4 * g], bh, bl);
        acc = mfma(w2[kk], bh, acc);
        acc = mfma(w2[kk], bl, acc);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) h2[i] = tanhf(acc[i]);
    }
    *(float4 *)&sZ[c * kRowH + u0] = make_float4(h2[0], h2[1], h2[2], h2[3]);
    __syncthreads();
    if (!TRAIN && wave > 0) continue;  // (every wave meets every barrier of every chunk)
    // output unit: lane (g, c) adds units 16 t + 4 g + i, then the four lanes of a column
    float z = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float4 q = *(const float4 *)&sZ[c * kRowH + 16 * t + 4 * g];
      z += w3[t][0] * q.x;
      z += w3[t][1] * q.y;
      z += w3[t][2] * q.z;
      z += w3[t][3] * q.w;
    }
    z += __shfl_xor(z, 16);
    z += __shfl_xor(z, 32);
    z += b3;
    const float yv = softplus(z);
    if (!TRAIN) {
      if (ok && g == 0) {
        if (y) y[s] = yv;
        if (nu) nu[s] = nu_scale * (double)yv;
      }
      continue;
    }
    // loss terms and dL/dz = 2 (y - t) / n * softplus'(z)
    const float r = ok ? yv - target : 0.f;
    const float dz = ok ? 2.f * r * inv_n * logistic(z) : 0.f;
    // delta2 = dz w3 (1 - h2^2)
    float d2[4], d1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) d2[i] = dz * w3u[i] * (1.f - h2[i] * h2[i]);
    put4(&sD2[c * kRowH + u0], d2);
    __syncthreads();
    // delta1 = (W2^T delta2) (1 - h1^2)
    {
      v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        v4s bh, bl;
        operand(&sD2[c * kRowH + 16 * kk + 4 * g], bh, bl);
        acc = mfma(w2t[kk], bh, acc);
        acc = mfma(w2t[kk], bl, acc);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) d1[i] = acc[i] * (1.f - h1[i] * h1[i]);
    }
    put4(&sD1[c * kRowH + u0], d1);
    // bias and output-weight sums over the 16 samples, on every lane of a row
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      vd1[i] += row_sum(d1[i]);
      vd2[i] += row_sum(d2[i]);
      vw3[i] += row_sum(dz * h2[i]);
    }
    vz += dz;
    vl += r * r;
    __syncthreads();
    // weight gradients of the chunk: the matrix product's K runs over its 16 samples
    v4s ah, al, bh, bl;
    operand_samples<kRowH>(sD1, g, 16 * wave + c, ah, al);
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      operand_samples<kRowX>(sX, g, 16 * t + c, bh, bl);
      gW1[t] = mfma(ah, bh, gW1[t]);
      gW1[t] = mfma(ah, bl, gW1[t]);
      gW1[t] = mfma(al, bh, gW1[t]);
    }
    operand_samples<kRowH>(sD2, g, 16 * wave + c, ah, al);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      operand_samples<kRowH>(sH1, g, 16 * t + c, bh, bl);
      gW2[t] = mfma(ah, bh, gW2[t]);
      gW2[t] = mfma(ah, bl, gW2[t]);
      gW2[t] = mfma(al, bh, gW2[t]);
    }
    __syncthreads();  // before the next chunk's samples
  }
  if (!TRAIN) return;
  float *out = part + (int64_t)blockIdx.x * (a.np + 1);
  // D[m][k]: lane holds rows 16 wave + 4 g + i, column 16 t + c
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = u0 + i;
#pragma unroll
    for (int t = 0; t < KT; ++t)
      if (16 * t + c < a.F) out[a.oW1 + (int64_t)m * a.F + 16 * t + c] = gW1[t][i];
#pragma unroll
    for (int t = 0; t < 4; ++t) out[a.oW2 + (int64_t)m * H + 16 * t + c] = gW2[t][i];
    if (c == 0) {
      out[a.ob1 + m] = vd1[i];
      out[a.ob2 + m] = vd2[i];
      out[a.ow3 + m] = vw3[i];
    }
  }
  vz = row_sum(vz);
  vl = row_sum(vl);
  if (threadIdx.x == 0) {
    out[a.ob3] = vz;
    out[a.np] = vl * inv_n;
  }
}

// bf16 copies of parameter i from its master value
__device__ __forceinline__ void write_copies(int64_t i, float th, int F, int FP, int64_t oW1, int64_t oW2,
                                             int64_t ow3, unsigned short *W1b, unsigned short *W2b,
                                             unsigned short *W2Tb, float *w3r) {
  if (i >= oW1 && i < oW1 + (int64_t)H * F) {
    const int64_t j = i - oW1;
    W1b[(j / F) * FP + j % F] = bf16_bits(th);
  } else if (i >= oW2 && i < oW2 + H * H) {
    const int j = (int)(i - oW2);
    const unsigned short b = bf16_bits(th);
    W2b[j] = b;
    W2Tb[(j % H) * H + j / H] = b;
  } else if (i >= ow3 && i < ow3 + H) {
    w3r[i - ow3] = bf16_val(bf16_bits(th));
  }
}

// Sum the partials in a fixed order (each of kAdamWays threads a run of them, in double:
// there are up to 256), eight loads in flight per thread;
// optionally export the gradient and the loss; optionally take one Adam step and refresh the bf16
// copies.
constexpr int kAdamWays = 8;
__global__ __launch_bounds__(64 * kAdamWays) void k_mlp_adam(const float *__restrict__ part, int parts, int64_t np,
                                                  float *__restrict__ grad, float *__restrict__ loss, int update,
                                                  float lr, float c1, float c2, float *__restrict__ theta,
                                                  float *__restrict__ am, float *__restrict__ av, int F, int FP,
                                                  int64_t oW1, int64_t oW2, int64_t ow3, unsigned short *W1b,
                                                  unsigned short *W2b, unsigned short *W2Tb, float *w3r) {
  __shared__ double sum[kAdamWays][64];
  const int64_t i = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
  const int way = threadIdx.x >> 6, each = (parts + kAdamWays - 1) / kAdamWays;
  const int from = way * each, to = from + each < parts ? from + each : parts;
  double q = 0.0;
  if (i <= np) {
#pragma unroll 8
    for (int s = from; s < to; ++s) q += part[(int64_t)s * (np + 1) + i];
  }
  sum[way][threadIdx.x & 63] = q;
  __syncthreads();
  if (way > 0 || i > np) return;
  double total = 0.0;
#pragma unroll
  for (int w = 0; w < kAdamWays; ++w) total += sum[w][threadIdx.x];
  const float gsum = (float)total;
  if (i == np) {
    if (loss) *loss = gsum;
    return;
  }
  if (grad) grad[i] = gsum;
  if (!update) return;
  const float m = 0.9f * am[i] + 0.1f * gsum;
  const float v = 0.999f * av[i] + 0.001f * gsum * gsum;
  am[i] = m;
  av[i] = v;
  const float th = theta[i] - lr * (m * c1) / (sqrtf(v * c2) + 1e-8f);
  theta[i] = th;
  write_copies(i, th, F, FP, oW1, oW2, ow3, W1b, W2b, W2Tb, w3r);
}

__global__ __launch_bounds__(256) void k_mlp_refresh(const float *__restrict__ theta, int64_t np, int F, int FP,
                                                     int64_t oW1, int64_t oW2, int64_t ow3, unsigned short *W1b,
                                                     unsigned short *W2b, unsigned short *W2Tb, float *w3r) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= np) return;
  write_copies(i, theta[i], F, FP, oW1, oW2, ow3, W1b, W2b, W2Tb, w3r);
}

}  // namespace

struct fr_mlp_s {
  uint64_t magic;
  Net net;
  hipStream_t stream;
  int device;
};

namespace {

constexpr uint64_t kMlpMagic = 0x46524d4c504e4554ull;  // "FRMLPNET"

bool valid(fr_mlp_t m) { return m && m->magic == kMlpMagic; }

#define MCHK(call)                                                                               \
  do {                                                                                           \
    hipError_t e_ = (call);                                                                      \
    if (e_ != hipSuccess) return fr_fail(FR_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

NetArgs args_of(const Net &n) {
  NetArgs a;
  a.F = n.F;
  a.FP = n.FP;
  a.W1b = n.W1b;
  a.W2b = n.W2b;
  a.W2Tb = n.W2Tb;
  a.b1 = n.theta + n.ob1;
  a.b2 = n.theta + n.ob2;
  a.w3r = n.w3r;
  a.b3 = n.theta + n.ob3;
  a.mean = n.mean;
  a.istd = n.istd;
  a.np = n.np;
  a.oW1 = n.oW1;
  a.ob1 = n.ob1;
  a.oW2 = n.oW2;
  a.ob2 = n.ob2;
  a.ow3 = n.ow3;
  a.ob3 = n.ob3;
  return a;
}

// Blocks of an evaluation: at most as many as the chip holds at once (by its registers a CU holds 6
// blocks of the kernel for up to 16 inputs, 5 up to 80, 4 above); they loop over the samples beyond,
// with their weights loaded once. Per sample a block for every 16 costs more than the wave for every
// 16 that loaded all the weights did where the inputs are few. 65536 samples (us), that wave / a
// block for every 16 / these blocks: 5 inputs 12.4 / 14.6 / 11.4, 31 15.0 / 17.4 / 15.2, 68
// 20.7 / 19.5 / 17.0, 128 40.2 / 33.0 / 22.8.
constexpr int64_t eval_blocks(int kt) { return 256 * (kt == 1 ? 6 : (kt <= 5 ? 5 : 4)); }

// Blocks of the training pass over n samples: one per 16 samples up to a block per CU.
constexpr int64_t train_parts(int64_t n) {
  const int64_t chunks = (n + kChunk - 1) / kChunk;
  return chunks < kMaxPart ? chunks : kMaxPart;
}

// part: the partial gradients of a training pass (the network's own or the fixed scratch array)
template <bool TRAIN>
int launch_mlp(const Net &net, hipStream_t st, const float *X, int64_t n, int64_t ldx, float *y, double *nu,
               double nu_scale, const float *tgt, float *part = nullptr) {
  const NetArgs a = args_of(net);
  const int64_t chunks = (n + kChunk - 1) / kChunk;
  const unsigned blocks = (unsigned)(TRAIN ? train_parts(n) : std::min(chunks, eval_blocks(net.FP / 16)));
  const float inv_n = 1.f / (float)n;
  switch (net.FP / 16) {
#define CASE(K)                                                                                                  \
  case K:                                                                                                        \
    hipLaunchKernelGGL((k_mlp<K, TRAIN>), dim3(blocks), dim3(256), 0, st, a, X, n, ldx, y, nu, nu_scale, tgt,   \
                       inv_n, part);                                                                             \
    break;
    CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
#undef CASE
    default: return fr_fail(FR_ERR_ARG, "network input size out of range");
  }
  MCHK(hipGetLastError());
  return FR_OK;
}

int ensure_scratch(Net &net, int64_t n) {
  const int64_t parts = train_parts(n);
  if (parts > net.part_cap) {
    if (net.part) (void)hipFree(net.part);
    net.part = nullptr;
    net.part_cap = 0;
    MCHK(hipMalloc(&net.part, parts * (net.np + 1) * sizeof(float)));
    net.part_cap = parts;
  }
  return FR_OK;
}

// forward + backward + gradient; then the Adam kernel (update or export only). fixed: training
// scratch to use instead of the network's own (which is grown here otherwise).
int grad_pass(fr_mlp_t m, const float *X, int64_t n, int64_t ldx, const float *t, bool update, float lr,
              float *loss_dev, float *fixed = nullptr) {
  Net &net = m->net;
  if (!X || !t || n <= 0 || ldx < net.F) return fr_fail(FR_ERR_ARG, "bad X / t / n / ldx");
  if (!fixed) {
    int rc = ensure_scratch(net, n);
    if (rc) return rc;
  }
  float *part = fixed ? fixed : net.part;
  int rc = launch_mlp<true>(net, m->stream, X, n, ldx, nullptr, nullptr, 0.0, t, part);
  if (rc) return rc;
  float c1 = 1.f, c2 = 1.f;
  if (update) {
    net.step += 1;
    c1 = (float)(1.0 / (1.0 - std::pow(0.9, net.step)));
    c2 = (float)(1.0 / (1.0 - std::pow(0.999, net.step)));
  }
  hipLaunchKernelGGL(k_mlp_adam, dim3((unsigned)((net.np + 1 + 63) / 64)), dim3(64 * kAdamWays), 0, m->stream, part,
                     (int)train_parts(n), net.np, update ? nullptr : net.grad, loss_dev, update ? 1 : 0, lr, c1, c2,
                     net.theta, net.am, net.av, net.F, net.FP, net.oW1, net.oW2, net.ow3, net.W1b, net.W2b,
                     net.W2Tb, net.w3r);
  MCHK(hipGetLastError());
  return FR_OK;
}

int upload_params(fr_mlp_t m, const float *params) {
  Net &net = m->net;
  MCHK(hipMemcpyAsync(net.theta, params, net.np * sizeof(float), hipMemcpyHostToDevice, m->stream));
  MCHK(hipMemsetAsync(net.am, 0, net.np * sizeof(float), m->stream));
  MCHK(hipMemsetAsync(net.av, 0, net.np * sizeof(float), m->stream));
  hipLaunchKernelGGL(k_mlp_refresh, dim3((unsigned)((net.np + 255) / 256)), dim3(256), 0, m->stream, net.theta,
                     net.np, net.F, net.FP, net.oW1, net.oW2, net.ow3, net.W1b, net.W2b, net.W2Tb, net.w3r);
  MCHK(hipGetLastError());
  MCHK(hipStreamSynchronize(m->stream));
  net.step = 0;
  return FR_OK;
}

void free_net(Net &n) {
  for (void *p : {(void *)n.theta, (void *)n.am, (void *)n.av, (void *)n.W1b, (void *)n.W2b, (void *)n.W2Tb,
                  (void *)n.w3r, (void *)n.mean, (void *)n.istd, (void *)n.part, (void *)n.grad, (void *)n.dloss})
    if (p) (void)hipFree(p);
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Training without allocation (fr_mlp_train_step_noalloc): the partial gradients of one call live
// in `scratch`, a fixed array each GPU holds for the life of the process, sized for
// kNoAllocMaxN samples at the largest input count. Host code never passes the array's name to a
// kernel (on the host it is only a stand-in for the symbol): each device's address comes from
// hipGetSymbolAddress, taken once per device with that device current, and is kept here.
// ------------------------------------------------------------------------------------------
namespace {

constexpr int64_t kNoAllocMaxN = FR_MLP_NOALLOC_MAX_N;
constexpr int64_t kMaxParams = (int64_t)H * kMaxIn + H + H * H + H + H + 1;
constexpr int64_t kScratchFloats = train_parts(kNoAllocMaxN) * (kMaxParams + 1);  // 12.2 MiB

}  // namespace

static __device__ __align__(256) float scratch[kScratchFloats];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_addr[kMaxDevices] = {};

// The device address of `scratch` on device dev (looked up once per device, that device made
// current for the lookup).
int scratch_address(int dev, float **out) {
  if (dev < 0 || dev >= kMaxDevices) return fr_fail(FR_ERR_UNSUPPORTED, "device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    int cur = -1;
    MCHK(hipGetDevice(&cur));
    if (cur != dev) MCHK(hipSetDevice(dev));
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != dev) (void)hipSetDevice(cur);
    if (e != hipSuccess || !p)
      return fr_fail(FR_ERR_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch_addr[dev] = (float *)p;
  }
  *out = g_scratch_addr[dev];
  return FR_OK;
}

}  // namespace

namespace frk {

int mlp_n_in(fr_mlp_t m) { return valid(m) ? m->net.F : -1; }

int mlp_forward_nu(fr_mlp_t m, const float *X, int64_t n, int64_t ldx, double *nu, double nu_scale,
                   void *stream) {
  if (!valid(m)) return fr_fail(FR_ERR_ARG, "invalid network handle");
  return launch_mlp<false>(m->net, (hipStream_t)stream, X, n, ldx, nullptr, nu, nu_scale, nullptr);
}

}  // namespace frk

extern "C" {

int64_t fr_mlp_n_params(int32_t n_in) { return (int64_t)H * n_in + H + H * H + H + H + 1; }

int fr_mlp_create(int32_t n_in, const float *params, const float *mean, const float *std_dev, void *hip_stream,
                  fr_mlp_t *out) {
  if (!out) return fr_fail(FR_ERR_ARG, "out is NULL");
  *out = nullptr;
  if (n_in < 1 || n_in > kMaxIn) return fr_fail(FR_ERR_ARG, "n_in must be in 1..128");
  if (!params || !mean || !std_dev) return fr_fail(FR_ERR_ARG, "params / mean / std is NULL");
  for (int k = 0; k < n_in; ++k)
    if (!(std_dev[k] > 0.f) || !std::isfinite(mean[k])) return fr_fail(FR_ERR_ARG, "std must be > 0, mean finite");
  const int64_t np = fr_mlp_n_params(n_in);
  for (int64_t i = 0; i < np; ++i)
    if (!std::isfinite(params[i])) return fr_fail(FR_ERR_ARG, "non-finite parameter");
  fr_mlp_s *m = new fr_mlp_s();
  m->magic = kMlpMagic;
  m->stream = (hipStream_t)hip_stream;
  (void)hipGetDevice(&m->device);
  Net &n = m->net;
  n.F = n_in;
  n.FP = (n_in + 15) / 16 * 16;
  n.np = np;
  n.oW1 = 0;
  n.ob1 = (int64_t)H * n_in;
  n.oW2 = n.ob1 + H;
  n.ob2 = n.oW2 + H * H;
  n.ow3 = n.ob2 + H;
  n.ob3 = n.ow3 + H;
  auto fail_free = [&](const std::string &msg) {
    free_net(n);
    delete m;
    return fr_fail(FR_ERR_HIP, msg);
  };
  if (hipMalloc(&n.theta, np * sizeof(float)) || hipMalloc(&n.am, np * sizeof(float)) ||
      hipMalloc(&n.av, np * sizeof(float)) || hipMalloc(&n.W1b, (size_t)H * n.FP * 2) ||
      hipMalloc(&n.W2b, H * H * 2) || hipMalloc(&n.W2Tb, H * H * 2) || hipMalloc(&n.w3r, H * sizeof(float)) ||
      hipMalloc(&n.mean, n.FP * sizeof(float)) || hipMalloc(&n.istd, n.FP * sizeof(float)) ||
      hipMalloc(&n.grad, np * sizeof(float)) || hipMalloc(&n.dloss, sizeof(float)))
    return fail_free("hipMalloc failed");
  std::vector<float> mp(n.FP, 0.f), ip(n.FP, 0.f);
  for (int k = 0; k < n_in; ++k) {
    mp[k] = mean[k];
    ip[k] = 1.f / std_dev[k];
  }
  if (hipMemcpy(n.mean, mp.data(), n.FP * sizeof(float), hipMemcpyHostToDevice) ||
      hipMemcpy(n.istd, ip.data(), n.FP * sizeof(float), hipMemcpyHostToDevice) ||
      hipMemset(n.W1b, 0, (size_t)H * n.FP * 2) || hipDeviceSynchronize())
    return fail_free("initial copies failed");
  int rc = upload_params(m, params);
  if (rc) {
    free_net(n);
    delete m;
    return rc;
  }
  *out = m;
  return FR_OK;
}

int fr_mlp_destroy(fr_mlp_t m) {
  if (!m) return FR_OK;
  if (!valid(m)) return fr_fail(FR_ERR_ARG, "invalid network handle");
  (void)hipStreamSynchronize(m->stream);
  free_net(m->net);
  m->magic = 0;
  delete m;
  return FR_OK;
}

int fr_mlp_set_stream(fr_mlp_t m, void *hip_stream) {
  if (!valid(m)) return fr_fail(FR_ERR_ARG, "invalid network handle");
  m->stream = (hipStream_t)hip_stream;
  return FR_OK;
}

int fr_mlp_set_params(fr_mlp_t m, const float *params) {
  if (!valid(m) || !params) return fr_fail(FR_ERR_ARG, "invalid network handle or params");
  for (int64_t i = 0; i < m->net.np; ++i)
    if (!std::isfinite(params[i])) return fr_fail(FR_ERR_ARG, "non-finite parameter");
  return upload_params(m, params);
}

int fr_mlp_get_params(fr_mlp_t m, float *params) {
  if (!valid(m) || !params) return fr_fail(FR_ERR_ARG, "invalid network handle or params");
  MCHK(hipMemcpyAsync(params, m->net.theta, m->net.np * sizeof(float), hipMemcpyDeviceToHost, m->stream));
  MCHK(hipStreamSynchronize(m->stream));
  return FR_OK;
}

int fr_mlp_get_bf16(fr_mlp_t m, uint16_t *W1, uint16_t *W2, uint16_t *w3) {
  if (!valid(m)) return fr_fail(FR_ERR_ARG, "invalid network handle");
  const Net &n = m->net;
  MCHK(hipStreamSynchronize(m->stream));
  if (W1) {
    std::vector<uint16_t> tmp((size_t)H * n.FP);
    MCHK(hipMemcpy(tmp.data(), n.W1b, tmp.size() * 2, hipMemcpyDeviceToHost));
    for (int r = 0; r < H; ++r)
      for (int k = 0; k < n.F; ++k) W1[r * n.F + k] = tmp[(size_t)r * n.FP + k];
  }
  if (W2) MCHK(hipMemcpy(W2, n.W2b, H * H * 2, hipMemcpyDeviceToHost));
  if (w3) {
    float tmp[H];
    MCHK(hipMemcpy(tmp, n.w3r, sizeof tmp, hipMemcpyDeviceToHost));
    for (int i = 0; i < H; ++i) {
      uint32_t u;
      std::memcpy(&u, &tmp[i], 4);
      w3[i] = (uint16_t)(u >> 16);
    }
  }
  return FR_OK;
}

int fr_mlp_forward(fr_mlp_t m, const float *X, int64_t n, int64_t ldx, float *y) {
  if (!valid(m)) return fr_fail(FR_ERR_ARG, "invalid network handle");
  if (n == 0) return FR_OK;
  if (!X || !y || n < 0 || ldx < m->net.F) return fr_fail(FR_ERR_ARG, "bad X / y / n / ldx");
  return launch_mlp<false>(m->net, m->stream, X, n, ldx, y, nullptr, 0.0, nullptr);
}

int fr_mlp_loss_grad(fr_mlp_t m, const float *X, int64_t n, int64_t ldx, const float *t, float *grad,
                     double *loss) {
  if (!valid(m)) return fr_fail(FR_ERR_ARG, "invalid network handle");
  int rc = grad_pass(m, X, n, ldx, t, false, 0.f, m->net.dloss);
  if (rc) return rc;
  if (grad) MCHK(hipMemcpyAsync(grad, m->net.grad, m->net.np * sizeof(float), hipMemcpyDeviceToHost, m->stream));
  float l = 0.f;
  MCHK(hipMemcpyAsync(&l, m->net.dloss, sizeof(float), hipMemcpyDeviceToHost, m->stream));
  MCHK(hipStreamSynchronize(m->stream));
  if (loss) *loss = l;
  return FR_OK;
}

int fr_mlp_train_step(fr_mlp_t m, const float *X, int64_t n, int64_t ldx, const float *t, float lr, float *loss) {
  if (!valid(m)) return fr_fail(FR_ERR_ARG, "invalid network handle");
  if (!(lr > 0.f)) return fr_fail(FR_ERR_ARG, "lr must be > 0");
  return grad_pass(m, X, n, ldx, t, true, lr, loss);
}

int fr_mlp_train_step_noalloc(fr_mlp_t m, const float *X, int64_t n, int64_t ldx, const float *t, float lr,
                              float *loss) {
  if (!valid(m)) return fr_fail(FR_ERR_ARG, "invalid network handle");
  if (!(lr > 0.f)) return fr_fail(FR_ERR_ARG, "lr must be > 0");
  if (n <= 0 || n > kNoAllocMaxN)
    return fr_fail(FR_ERR_ARG, "n must be in 1.." + std::to_string(kNoAllocMaxN) + " for the no-allocation step");
  const Net &net = m->net;
  if (train_parts(n) * (net.np + 1) > kScratchFloats) return fr_fail(FR_ERR_ARG, "batch exceeds the scratch array");
  float *base = nullptr;
  int rc = scratch_address(m->device, &base);
  if (rc) return rc;
  // (every entry of the partial gradients that the Adam kernel reads is first written by this call)
  return grad_pass(m, X, n, ldx, t, true, lr, loss, base);
}

}  // extern "C"
