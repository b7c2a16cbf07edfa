// Learned warm start: a small MLP (features -> SiLU hidden layers -> linear
// output) evaluated with BF16 MFMA (FP32 accumulate), trained with FP32
// backward kernels and Adam, plus the conversions between the solver's
// state arena and the network's features / targets / outputs.
//
// Parameter layout (padded, shared by the BF16 copy, the FP32 master copy,
// Adam moments and gradients): for layer l = 0 .. n_hidden, W_l as [N_l][K_l]
// (output-major) followed by b_l [N_l], with K_0 = 16 (inputs zero-padded),
// K_l = N_l = d_hidden for hidden-to-hidden layers and N_out = 16 (outputs
// zero-padded).  Padded weights start at zero and receive zero gradients, so
// they stay zero.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "cfd_internal.hpp"

namespace cfd {

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));
// the same in the caller's memory, which is aligned to its elements only
typedef short4_t short4_mem __attribute__((aligned(2)));
typedef short short8_t __attribute__((ext_vector_type(8)));
typedef short8_t short8_mem __attribute__((aligned(2)));
typedef float4_t float4_mem __attribute__((aligned(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {   // round to nearest even
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// 4 floats -> 4 BF16, nearest even (v_cvt_pk_bf16_f32)
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ short4_t pack_bf16(float4_t f) {
  return __builtin_bit_cast(short4_t, __builtin_convertvector(f, bf16x4));
}
__device__ __forceinline__ float4_t unpack_bf16(short4_t h) {
  return float4_t{bf2f((uint16_t)h[0]), bf2f((uint16_t)h[1]), bf2f((uint16_t)h[2]), bf2f((uint16_t)h[3])};
}

// SiLU and its derivative, by the general division (infinities, NaN and quotients
// below the normal range included).
__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_grad_f(float z) {
  const float s = 1.0f / (1.0f + __expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// silu_f's value to the bit (but for the sign of zero) where |z| < SILU_MID, the
// denominator in [1, 2^100): reciprocal estimate, one Newton-Raphson step,
// quotient, two residual corrections q' = q + r (z - d q) (Markstein, IBM J. Res.
// Dev. 34(1), 1990), without the scaling and the special cases of the general
// division.  For large batches, where SiLU is what bounds the pass: 1,769,472
// points of the 5-128x4-5 net 0.494 ms, 0.537 with the division alone.  A wave of
// small batches has its SIMD to itself, and the branch costs it more than the
// division (131,071 points: 76 us against 63).
constexpr float SILU_MID = 69.0f;
__device__ __forceinline__ float silu_mid(float z) {
  const float d = 1.0f + __expf(-z);
  float r = __builtin_amdgcn_rcpf(d);
  r = __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
  float q = z * r;
  q = __builtin_fmaf(__builtin_fmaf(-d, q, z), r, q);
  return __builtin_fmaf(__builtin_fmaf(-d, q, z), r, q);
}

// ------------------------------------------------------------------ forward
// Activations stay in registers.  A layer is D = W X with the weights as the
// MFMA's A operand and 16 points as its columns, whose layouts are
//   A (16 outputs x 16 k): lane l holds row l%16,   k = 4 (l/16) .. +3
//   B (16 k x 16 points):  lane l holds column l%16, k = 4 (l/16) .. +3
//   D (16 outputs x 16 points): lane l holds rows 4 (l/16) .. +3, column l%16
// so a D tile, through SiLU and rounded to BF16, is the next layer's B tile as
// it stands.  The weights lie in LDS in A-fragment order (8 bytes a lane, 512
// contiguous bytes a tile: no bank conflicts), the whole net at once where it
// fits (staged once by each workgroup of a persistent grid), else layer by
// layer.  A wave takes M tiles of 16 points, so that one weight fragment feeds
// M MFMAs.
//
// Bound: SiLU (exp and reciprocal at a quarter of the VALU rate, about 80 issue
// cycles a wave and activation) before the MFMAs (106 kflop a point).
// 1,769,472 points of the 5-128x4-5 net: 0.494 ms (0.380 PFLOP/s); 2.45 ms with
// the activations in LDS and the weights read from L2 by every wave.
constexpr int MLP_LDS_MAX = 144 * 1024;   // weights held by a workgroup

struct MlpStage {   // LDS elements (uint16) of a layer's fragments and its biases (float)
  int frag[MLP_MAX_LAYERS], bias[MLP_MAX_LAYERS];
  int bytes;        // of the whole net, or of the largest layer
  int resident;     // 1: the whole net is in LDS
};

// Layer l's weights (NT x KT tiles) -> fragment order at w, its biases -> b (all
// threads of the workgroup).  16-byte loads, eight of a thread in flight.
template <int KT, int NT>
__device__ __forceinline__ void stage_layer(const MlpDims& D, int l, const uint16_t* __restrict__ P, uint16_t* w,
                                            float* b) {
  constexpr int K = KT * 16;
  const uint16_t* W = P + D.woff[l];
#pragma unroll 8
  for (int e = threadIdx.x; e < NT * 16 * K / 8; e += blockDim.x) {   // 8 consecutive k of a row
    const int row = e / (K / 8), k = (e - row * (K / 8)) * 8;
    const short8_t v = *reinterpret_cast<const short8_mem*>(W + (int64_t)row * K + k);
    uint16_t* at = w + (((row >> 4) * KT + (k >> 4)) * 64 + (row & 15) + 16 * ((k >> 2) & 3)) * 4;
    *reinterpret_cast<short4_t*>(at) = __builtin_shufflevector(v, v, 0, 1, 2, 3);
    *reinterpret_cast<short4_t*>(at + 64) = __builtin_shufflevector(v, v, 4, 5, 6, 7);
  }
  for (int e = threadIdx.x; e < NT * 16; e += blockDim.x) b[e] = bf2f(P[D.boff[l] + e]);
}

// One layer of KT input tiles and NT output tiles.  in: B fragments; out: the
// next layer's B fragments, or with last the outputs' D tile in y.
template <int KT, int NT, int M, bool CACHE, bool LAST>
__device__ __forceinline__ void layer_fwd(const uint16_t* w, const float* b, const short4_t (&in)[M][KT],
                                          short4_t (&out)[M][NT], float4_t (&y)[M], const int64_t (&p)[M], int64_t n,
                                          float* __restrict__ cache, int64_t cpp, int64_t zoff, int64_t hoff) {
  const int lane = threadIdx.x & 63, g4 = (lane >> 4) * 4;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float4_t acc[M];
#pragma unroll
    for (int m = 0; m < M; ++m) acc[m] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KT; ++ks) {
      const short4_t a = *reinterpret_cast<const short4_t*>(w + ((nt * KT + ks) * 64 + lane) * 4);
#pragma unroll
      for (int m = 0; m < M; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, in[m][ks], acc[m], 0, 0, 0);
    }
    const float4_t bias = *reinterpret_cast<const float4_t*>(b + nt * 16 + g4);
    float most = 0.f;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      acc[m] = acc[m] + bias;
      if (CACHE && p[m] < n) *reinterpret_cast<float4_mem*>(cache + p[m] * cpp + zoff + nt * 16 + g4) = acc[m];
      if (LAST) y[m] = acc[m];
#pragma unroll
      for (int r = 0; r < 4; ++r) most = fmaxf(most, fabsf(acc[m][r]));
    }
    if (LAST) continue;
    if (M == 1 || __any(most >= SILU_MID)) {
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[m][r] = silu_f(acc[m][r]);
    } else {
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[m][r] = silu_mid(acc[m][r]);
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      out[m][nt] = pack_bf16(acc[m]);
      if (CACHE && p[m] < n)
        *reinterpret_cast<float4_mem*>(cache + p[m] * cpp + hoff + nt * 16 + g4) = unpack_bf16(out[m][nt]);
    }
  }
}

template <int HT, int M, bool CACHE, int NT>
__global__ void __launch_bounds__(NT) k_mlp_forward(MlpDims D, MlpStage S, const uint16_t* __restrict__ P,
                                                    const float* __restrict__ x, const int32_t* __restrict__ idx,
                                                    int64_t n, float* __restrict__ y, float* __restrict__ cache) {
  extern __shared__ __attribute__((aligned(16))) char mlp_lds[];
  uint16_t* const lw = reinterpret_cast<uint16_t*>(mlp_lds);
  float* const lb = reinterpret_cast<float*>(mlp_lds);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g4 = (lane >> 4) * 4;
  constexpr int PTS = NT / 64 * M * 16;     // points of a workgroup's round
  const int64_t cpp = D.cache_per_point;
  const int last = D.nlayer - 1;
  if (S.resident) {
    stage_layer<1, HT>(D, 0, P, lw + S.frag[0], lb + S.bias[0]);
    for (int l = 1; l < last; ++l) stage_layer<HT, HT>(D, l, P, lw + S.frag[l], lb + S.bias[l]);
    stage_layer<HT, 1>(D, last, P, lw + S.frag[last], lb + S.bias[last]);
    __syncthreads();
  }
  // every wave of a workgroup takes the same rounds (the layer-by-layer path has barriers)
  for (int64_t p0 = (int64_t)blockIdx.x * PTS; p0 < n; p0 += (int64_t)gridDim.x * PTS) {
    int64_t p[M];
    short4_t x0[M][1], h[M][HT];
    float4_t yo[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      p[m] = p0 + (wave * M + m) * 16 + (lane & 15);
      float4_t v = {0.f, 0.f, 0.f, 0.f};
      if (p[m] < n) {
        const int64_t src = idx ? (int64_t)idx[p[m]] : p[m];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (g4 + r < D.d_in) v[r] = x[src * D.d_in + g4 + r];
      }
      x0[m][0] = pack_bf16(v);
      if (CACHE && p[m] < n)
        *reinterpret_cast<float4_mem*>(cache + p[m] * cpp + D.hoff[0] + g4) = unpack_bf16(x0[m][0]);
    }
    auto weights = [&](int l) {
      if (S.resident) return;
      __syncthreads();     // the previous layer's readers are done
      if (l == 0) stage_layer<1, HT>(D, l, P, lw + S.frag[l], lb + S.bias[l]);
      else if (l < last) stage_layer<HT, HT>(D, l, P, lw + S.frag[l], lb + S.bias[l]);
      else stage_layer<HT, 1>(D, l, P, lw + S.frag[l], lb + S.bias[l]);
      __syncthreads();
    };
    weights(0);
    layer_fwd<1, HT, M, CACHE, false>(lw + S.frag[0], lb + S.bias[0], x0, h, yo, p, n, cache, cpp, D.zoff[0],
                                      D.hoff[1]);
    for (int l = 1; l < last; ++l) {
      short4_t o[M][HT];
      weights(l);
      layer_fwd<HT, HT, M, CACHE, false>(lw + S.frag[l], lb + S.bias[l], h, o, yo, p, n, cache, cpp, D.zoff[l],
                                         D.hoff[l + 1]);
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int t = 0; t < HT; ++t) h[m][t] = o[m][t];
    }
    short4_t none[M][1];
    weights(last);
    layer_fwd<HT, 1, M, CACHE, true>(lw + S.frag[last], lb + S.bias[last], h, none, yo, p, n, cache, cpp,
                                     D.zoff[last], 0);
#pragma unroll
    for (int m = 0; m < M; ++m)
      if (p[m] < n)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (g4 + r < D.d_out) y[p[m] * D.d_out + g4 + r] = yo[m][r];
  }
}

// ------------------------------------------------------------------ loss
// dy = 2 (y - t) / (n d_out) on the d_out outputs; per-workgroup loss
// partials (fixed-order tree) for a deterministic mean squared error.
__global__ void __launch_bounds__(256) k_mlp_mse(const float* __restrict__ y, const float* __restrict__ t,
                                                 const int32_t* __restrict__ idx, int64_t n, int d_out,
                                                 float* __restrict__ dy, double* __restrict__ partials) {
  __shared__ double red[256];
  double acc = 0.0;
  const int64_t total = n * d_out;
  const float scale = 2.0f / (float)total;
  for (int64_t e = blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int64_t p = e / d_out;
    const int o = (int)(e - p * d_out);
    const int64_t src = idx ? (int64_t)idx[p] : p;
    const float d = y[e] - t[src * d_out + o];
    dy[e] = scale * d;
    acc += (double)d * (double)d;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partials[blockIdx.x] = red[0];
}

// The loss from the partials: a fixed tree over one workgroup.
__global__ void __launch_bounds__(256) k_mlp_mse_final(const double* __restrict__ partials, int nrows, int64_t count,
                                                       double* __restrict__ loss) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int r = threadIdx.x; r < nrows; r += 256) acc += partials[r];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[0] = red[0] / (double)count;
}

// ------------------------------------------------------------------ backward
// dZ_l (the loss gradient at layer l's pre-activation) of every layer, then all
// weight gradients dW_l = dZ_l^T H_l as one launch of split contractions, then
// their sum.  The contractions run on the BF16 MFMA at FP32 precision: the
// weights and the layer inputs H are BF16 values as they stand, and the FP32
// dZ is cut into three BF16 terms that add up to it (8 + 8 + 8 bits), so every
// product is exact and the accumulation is FP32.  Error of a layer's gradients
// against 64 bits at 8192 points: 3e-8 to 6e-8 of their norm (8e-8 to 1.3e-7
// with the scalar FP32 sums it replaces).
//
// A minibatch of 8192 through the 5-128x4-5 net: k_mlp_dz 31 us, k_mlp_dw 25,
// the sum 5; before, one thread per weight walked 256 points (547 us) and one
// per point and input summed dZ W (178 us), in 21 launches.  Latency bounds the
// new ones: 8192 points are half a wave a SIMD.
struct Split3 {
  short4_t hi, mid, lo;
};
// An infinity goes into mid (hi the largest BF16 value, lo zero), so that products
// and sums stay infinite, and a value past the largest BF16 one is not rounded to
// infinity.  Terms below BF16's least subnormal, 9e-41, are lost: values under
// 1e-33 have fewer than 24 bits.
__device__ __forceinline__ Split3 split3(float4_t v) {
  constexpr float BF16_MAX = 3.38953139e38f;
  Split3 s;
  float4_t c;
#pragma unroll
  for (int r = 0; r < 4; ++r) c[r] = __builtin_amdgcn_fmed3f(v[r], -BF16_MAX, BF16_MAX);
  s.hi = pack_bf16(c);
  v = v - unpack_bf16(s.hi);
  s.mid = pack_bf16(v);
  c = v - unpack_bf16(s.mid);
#pragma unroll
  for (int r = 0; r < 4; ++r) c[r] = __builtin_isinf(v[r]) ? 0.f : c[r];
  s.lo = pack_bf16(c);
  return s;
}
__device__ __forceinline__ float4_t mfma3(short4_t w, const Split3& d, float4_t acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w, d.lo, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w, d.mid, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w, d.hi, acc, 0, 0, 0);
}

// dZ of every layer, transposed: dzT[off[l] + o np + p], np points (n rounded up
// to 64; rows of the padding are zero).  A wave carries 16 points down the
// layers: dZ_l is the MFMA's B operand with the layout the product comes out in
// (as in the forward pass), W_l^T the A operand, staged in LDS in fragment order.
struct MlpDz {
  int64_t off[MLP_MAX_LAYERS], np;
};

template <int V>
struct Tiles {
  static constexpr int value = V;
};

template <int HT>
__global__ void __launch_bounds__(256) k_mlp_dz(MlpDims D, MlpDz Z, const uint16_t* __restrict__ P,
                                                const float* __restrict__ cache, const float* __restrict__ dy,
                                                int64_t n, float* __restrict__ dzT) {
  __shared__ __attribute__((aligned(16))) uint16_t sw[HT * HT * 256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g4 = (lane >> 4) * 4;
  const int64_t p = (int64_t)blockIdx.x * 64 + wave * 16 + (lane & 15);
  const int last = D.nlayer - 1;
  // W_l (NT x HT tiles) -> A fragments of W_l^T: tile (kt, t), lane l: row k = 16 kt + l%16, o = 16 t + 4 (l/16) .. +3
  auto stage = [&](int l, auto tiles) {
    constexpr int NT = decltype(tiles)::value, K = HT * 16;
    const uint16_t* W = P + D.woff[l];
#pragma unroll 8
    for (int e = threadIdx.x; e < NT * 16 * K / 8; e += 256) {
      const int o = e / (K / 8), k = (e - o * (K / 8)) * 8;
      const short8_t v = *reinterpret_cast<const short8_mem*>(W + (int64_t)o * K + k);
      uint16_t* at = sw + ((((k >> 4) * NT + (o >> 4)) * 64 + (k & 15) + 16 * ((o >> 2) & 3)) * 4 + (o & 3));
#pragma unroll
      for (int c = 0; c < 8; ++c) at[4 * c] = (uint16_t)v[c];
    }
  };
  auto store = [&](int l, int t, float4_t dz) {
#pragma unroll
    for (int r = 0; r < 4; ++r) dzT[Z.off[l] + (int64_t)(t * 16 + g4 + r) * Z.np + p] = dz[r];
  };
  // silu'(z_l) of every tile, loaded ahead of the layer's product
  auto grads = [&](int l, float4_t (&z)[HT]) {
#pragma unroll
    for (int t = 0; t < HT; ++t)
      z[t] = *reinterpret_cast<const float4_mem*>(cache + min(p, n - 1) * D.cache_per_point + D.zoff[l] + t * 16 + g4);
  };
  auto through = [&](int l, int kt, float4_t acc, float4_t z) {
    float4_t dz;
#pragma unroll
    for (int r = 0; r < 4; ++r) dz[r] = p < n ? acc[r] * silu_grad_f(z[r]) : 0.f;
    store(l, kt, dz);
    return split3(dz);
  };
  float4_t z[HT];
  grads(last - 1, z);
  float4_t out = {0.f, 0.f, 0.f, 0.f};
  if (p < n)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (g4 + r < D.d_out) out[r] = dy[p * D.d_out + g4 + r];
  store(last, 0, out);
  const Split3 so = split3(out);
  Split3 d[HT];
  stage(last, Tiles<1>{});
  __syncthreads();
#pragma unroll
  for (int kt = 0; kt < HT; ++kt) {
    const short4_t w = *reinterpret_cast<const short4_t*>(sw + (kt * 64 + lane) * 4);
    d[kt] = through(last - 1, kt, mfma3(w, so, float4_t{0.f, 0.f, 0.f, 0.f}), z[kt]);
  }
  for (int l = last - 1; l > 0; --l) {
    grads(l - 1, z);
    __syncthreads();
    stage(l, Tiles<HT>{});
    __syncthreads();
    Split3 e[HT];
    // pairs of tiles, so that two chains of MFMAs are in flight
#pragma unroll
    for (int kt = 0; kt < HT; kt += 2) {
      constexpr int last_t = HT - 1;
      const int k1 = kt < last_t ? kt + 1 : kt;
      float4_t a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < HT; ++t) {
        const short4_t w0 = *reinterpret_cast<const short4_t*>(sw + ((kt * HT + t) * 64 + lane) * 4);
        const short4_t w1 = *reinterpret_cast<const short4_t*>(sw + ((k1 * HT + t) * 64 + lane) * 4);
        a0 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w0, d[t].lo, a0, 0, 0, 0);
        a1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w1, d[t].lo, a1, 0, 0, 0);
        a0 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w0, d[t].mid, a0, 0, 0, 0);
        a1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w1, d[t].mid, a1, 0, 0, 0);
        a0 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w0, d[t].hi, a0, 0, 0, 0);
        a1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w1, d[t].hi, a1, 0, 0, 0);
      }
      e[kt] = through(l - 1, kt, a0, z[kt]);
      if (k1 != kt) e[k1] = through(l - 1, k1, a1, z[k1]);
    }
#pragma unroll
    for (int t = 0; t < HT; ++t) d[t] = e[t];
  }
}

// Weight and bias gradients of points [split chunk, ...): one wave per 32 x 32
// tile of one layer's dW and split, into part[split][nparam].  Bound by the
// latency of its gathers of 4.2 KB-apart cache rows, so smaller tiles (more
// waves) beat the reuse of larger ones: a minibatch of 8192 takes 88 us in all
// with 32 x 32, 92 with 32 x 64, 97 with 64 x 64.
constexpr int MLP_DW_O = 2, MLP_DW_K = 2;   // 16-wide tiles of a wave along outputs and inputs
__host__ __device__ inline int mlp_dw_tiles(int N, int K) {
  return ((N / 16 + MLP_DW_O - 1) / MLP_DW_O) * ((K / 16 + MLP_DW_K - 1) / MLP_DW_K);
}

__global__ void __launch_bounds__(64) k_mlp_dw(MlpDims D, MlpDz Z, const float* __restrict__ dzT,
                                               const float* __restrict__ cache, int64_t n, int64_t chunk,
                                               float* __restrict__ part) {
  const int lane = threadIdx.x, l16 = lane & 15, g4 = (lane >> 4) * 4;
  int l = 0, job = blockIdx.x;
  for (; job >= mlp_dw_tiles(D.N[l], D.K[l]); ++l) job -= mlp_dw_tiles(D.N[l], D.K[l]);
  const int N = D.N[l], K = D.K[l], kb = (K / 16 + MLP_DW_K - 1) / MLP_DW_K;
  const int o0 = (job / kb) * MLP_DW_O, k0 = (job % kb) * MLP_DW_K;
  const int no = min(MLP_DW_O, N / 16 - o0), nk = min(MLP_DW_K, K / 16 - k0);
  const int64_t pa = blockIdx.y * chunk, pb = min(Z.np, pa + chunk);
  const float* A = dzT + Z.off[l] + (int64_t)(o0 * 16 + l16) * Z.np + g4;
  const float* H = cache + D.hoff[l] + k0 * 16 + l16;
  float4_t acc[MLP_DW_O][MLP_DW_K] = {};
  float bias[MLP_DW_O] = {};
#pragma unroll 4
  for (int64_t p = pa; p < pb; p += 16) {
    short4_t h[MLP_DW_K];
#pragma unroll
    for (int kt = 0; kt < MLP_DW_K; ++kt) {
      float4_t v = {0.f, 0.f, 0.f, 0.f};
      if (kt < nk)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = H[min(p + g4 + c, n - 1) * D.cache_per_point + kt * 16];
      h[kt] = pack_bf16(v);     // H holds BF16 values: exact
    }
#pragma unroll
    for (int ot = 0; ot < MLP_DW_O; ++ot) {
      if (ot >= no) continue;
      const float4_t a = *reinterpret_cast<const float4_mem*>(A + (int64_t)ot * 16 * Z.np + p);
      bias[ot] += (a[0] + a[1]) + (a[2] + a[3]);
      const Split3 s = split3(a);
#pragma unroll
      for (int kt = 0; kt < MLP_DW_K; ++kt) {
        acc[ot][kt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(s.lo, h[kt], acc[ot][kt], 0, 0, 0);
        acc[ot][kt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(s.mid, h[kt], acc[ot][kt], 0, 0, 0);
        acc[ot][kt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(s.hi, h[kt], acc[ot][kt], 0, 0, 0);
      }
    }
  }
  float* out = part + (int64_t)blockIdx.y * D.nparam;
#pragma unroll
  for (int ot = 0; ot < MLP_DW_O; ++ot) {
    if (ot >= no) continue;
#pragma unroll
    for (int kt = 0; kt < MLP_DW_K; ++kt)
      if (kt < nk)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          out[D.woff[l] + (int64_t)((o0 + ot) * 16 + g4 + r) * K + (k0 + kt) * 16 + l16] = acc[ot][kt][r];
    float b = bias[ot];
    b += __shfl_xor(b, 16, 64);
    b += __shfl_xor(b, 32, 64);
    if (k0 == 0 && lane < 16) out[D.boff[l] + (o0 + ot) * 16 + lane] = b;
  }
}

// Sum of the splits, in order and in FP64 (an FP32 sum of 64 splits would cost
// the gradients a third of their last digit: 1.2e-7 against 0.95e-7 with the
// 32 longer FP32 sums it replaces).
__global__ void __launch_bounds__(256) k_mlp_dw_reduce(const float* __restrict__ part, int nsplit, int64_t np,
                                                       float* __restrict__ grad) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= np) return;
  double s = 0.0;
#pragma unroll 8
  for (int c = 0; c < nsplit; ++c) s += (double)part[c * np + e];
  grad[e] = (float)s;
}

// ------------------------------------------------------------------ Adam
__global__ void k_mlp_adam(int64_t np, float* __restrict__ master, float* __restrict__ m, float* __restrict__ v,
                           const float* __restrict__ g, uint16_t* __restrict__ pbf, float lr, float b1, float b2,
                           float eps, float c1, float c2) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= np) return;
  const float ge = g[e];
  const float me = b1 * m[e] + (1.f - b1) * ge;
  const float ve = b2 * v[e] + (1.f - b2) * ge * ge;
  m[e] = me;
  v[e] = ve;
  const float th = master[e] - lr * (me / c1) / (sqrtf(ve / c2) + eps);
  master[e] = th;
  pbf[e] = f2bf(th);
}

__global__ void k_mlp_to_bf16(int64_t np, const float* __restrict__ master, uint16_t* __restrict__ pbf) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e < np) pbf[e] = f2bf(master[e]);
}

// ------------------------------------------------------------ state <-> features
// Interior cells of all blocks in order (block, k, j, i); thread per cell.
// Features: [(M - 0.675)/0.175, (h - 0.06)/0.04, 2 xi - 1, 2 eta - 1, 2 zeta - 1].
__device__ __forceinline__ int find_block(const CellMap& M, int64_t e) {
  int lo = 0, hi = M.nblk - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (M.cell_start[mid] <= e) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

__global__ void k_mlp_features(CellMap M, int64_t ncells, const double* __restrict__ cond, float* __restrict__ x) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= ncells) return;
  const int b = find_block(M, e);
  const BlockDesc B = M.blocks[b];
  const int64_t r = e - M.cell_start[b];
  const int ni = B.n[0], nj = B.n[1], nk = B.n[2];
  const int i = (int)(r % ni), j = (int)((r / ni) % nj), k = (int)(r / ((int64_t)ni * nj));
  float* o = x + e * 5;
  o[0] = (float)((cond[2 * b] - 0.675) / 0.175);
  o[1] = (float)((cond[2 * b + 1] - 0.06) / 0.04);
  o[2] = (float)(2.0 * (i + 0.5) / ni - 1.0);
  o[3] = (float)(2.0 * (j + 0.5) / nj - 1.0);
  o[4] = (float)(2.0 * (k + 0.5) / nk - 1.0);
}

// Targets: primitive deviations from each block's inflow stream.
__global__ void k_mlp_targets(CellMap M, int64_t ncells, const double* __restrict__ q,
                              const double* __restrict__ cond, double gamma, float* __restrict__ t) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= ncells) return;
  const int b = find_block(M, e);
  const BlockDesc B = M.blocks[b];
  const int64_t r = e - M.cell_start[b];
  const int ni = B.n[0], nj = B.n[1];
  const int i = (int)(r % ni), j = (int)((r / ni) % nj), k = (int)(r / ((int64_t)ni * nj));
  const int64_t c = B.qoff + (int64_t)(k + NG) * B.sk + (int64_t)(j + NG) * B.sj + (i + NG);
  const double rho = q[c], inv = 1.0 / rho;
  const double u = q[B.sv + c] * inv, v = q[2 * B.sv + c] * inv, w = q[3 * B.sv + c] * inv;
  const double p = (gamma - 1.0) * (q[4 * B.sv + c] - 0.5 * rho * (u * u + v * v + w * w));
  float* o = t + e * 5;
  o[0] = (float)(rho - 1.0);
  o[1] = (float)(u - cond[2 * b] * sqrt(gamma));
  o[2] = (float)v;
  o[3] = (float)w;
  o[4] = (float)(p - 1.0);
}

// Network outputs -> conserved state of the interior cells (FP64).
__global__ void k_mlp_to_state(CellMap M, int64_t ncells, const float* __restrict__ yv,
                               const double* __restrict__ cond, double gamma, double* __restrict__ q) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= ncells) return;
  const int b = find_block(M, e);
  const BlockDesc B = M.blocks[b];
  const int64_t r = e - M.cell_start[b];
  const int ni = B.n[0], nj = B.n[1];
  const int i = (int)(r % ni), j = (int)((r / ni) % nj), k = (int)(r / ((int64_t)ni * nj));
  const int64_t c = B.qoff + (int64_t)(k + NG) * B.sk + (int64_t)(j + NG) * B.sj + (i + NG);
  const float* o = yv + e * 5;
  const double rho = 1.0 + (double)o[0];
  const double u = cond[2 * b] * sqrt(gamma) + (double)o[1];
  const double v = (double)o[2], w = (double)o[3];
  const double p = 1.0 + (double)o[4];
  q[c] = rho;
  q[B.sv + c] = rho * u;
  q[2 * B.sv + c] = rho * v;
  q[3 * B.sv + c] = rho * w;
  q[4 * B.sv + c] = p / (gamma - 1.0) + 0.5 * rho * (u * u + v * v + w * w);
}

// ------------------------------------------------------------------ launchers

static unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

// LDS plan of the net's weights: 8 bytes a lane and tile, biases as floats.
static MlpStage mlp_stage(const MlpDims& D) {
  MlpStage S{};
  int at = 0, most = 0;
  for (int l = 0; l < D.nlayer; ++l) {
    const int w = D.N[l] * D.K[l] * 2, b = D.N[l] * 4;
    S.frag[l] = at / 2;
    S.bias[l] = (at + w) / 4;
    at += w + b;
    most = std::max(most, w + b);
  }
  S.resident = at <= MLP_LDS_MAX;
  S.bytes = S.resident ? at : most;
  if (!S.resident)
    for (int l = 0; l < D.nlayer; ++l) {
      S.frag[l] = 0;
      S.bias[l] = D.N[l] * D.K[l] / 2;
    }
  return S;
}

template <int HT, int M, bool CACHE, int NT>
static void forward_launch(const MlpDims& D, const MlpStage& S, const uint16_t* P, const float* x, const int32_t* idx,
                           int64_t n, float* y, float* cache, hipStream_t s) {
  constexpr int PTS = NT / 64 * M * 16;
  const int64_t rounds = (n + PTS - 1) / PTS;
  // one workgroup a CU where each stages the whole net (a wide net fills its LDS; a
  // narrow one would hold more)
  const unsigned nwg = (unsigned)std::min<int64_t>(rounds, S.resident ? 256 : 1024);
  hipFuncSetAttribute(reinterpret_cast<const void*>(&k_mlp_forward<HT, M, CACHE, NT>),
                      hipFuncAttributeMaxDynamicSharedMemorySize, S.bytes);
  hipLaunchKernelGGL((k_mlp_forward<HT, M, CACHE, NT>), dim3(nwg), dim3(NT), S.bytes, s, D, S, P, x, idx, n, y, cache);
}

// Large batches: 16 waves of 32 points (a weight fragment feeds two MFMAs);
// batches that would leave CUs idle so, and training's (which also store every
// activation): 4 waves of 16 points.
template <int HT>
static void forward_width(const MlpDims& D, const MlpStage& S, const uint16_t* P, const float* x, const int32_t* idx,
                          int64_t n, float* y, float* cache, hipStream_t s) {
  if (cache) forward_launch<HT, 1, true, 256>(D, S, P, x, idx, n, y, cache, s);
  else if (n >= 256 * 512) forward_launch<HT, 2, false, 1024>(D, S, P, x, idx, n, y, cache, s);
  else forward_launch<HT, 1, false, 256>(D, S, P, x, idx, n, y, cache, s);
}

void mlp_forward(const MlpDims& D, const uint16_t* P, const float* x, const int32_t* idx, int64_t n, float* y,
                 float* cache, hipStream_t s) {
  const MlpStage S = mlp_stage(D);
  switch (D.d_hidden / 16) {
    case 1: return forward_width<1>(D, S, P, x, idx, n, y, cache, s);
    case 2: return forward_width<2>(D, S, P, x, idx, n, y, cache, s);
    case 3: return forward_width<3>(D, S, P, x, idx, n, y, cache, s);
    case 4: return forward_width<4>(D, S, P, x, idx, n, y, cache, s);
    case 5: return forward_width<5>(D, S, P, x, idx, n, y, cache, s);
    case 6: return forward_width<6>(D, S, P, x, idx, n, y, cache, s);
    case 7: return forward_width<7>(D, S, P, x, idx, n, y, cache, s);
    default: return forward_width<8>(D, S, P, x, idx, n, y, cache, s);
  }
}

int mlp_mse(const float* y, const float* t, const int32_t* idx, int64_t n, int d_out, float* dy, double* partials,
            int max_rows, double* loss, hipStream_t s) {
  int nb = (int)std::min<int64_t>(max_rows, std::max<int64_t>(1, (n * d_out + 255) / 256));
  hipLaunchKernelGGL(k_mlp_mse, dim3(nb), dim3(256), 0, s, y, t, idx, n, d_out, dy, partials);
  hipLaunchKernelGGL(k_mlp_mse_final, dim3(1), dim3(256), 0, s, partials, nb, n * d_out, loss);
  return nb;
}

// Splits of the weight gradients' points: 128 points each (8 MFMA steps; 256
// points a split, half the waves, cost a minibatch of 8192 6 to 13 us more), at
// most MLP_SPLITS.
int mlp_splits(int64_t n) { return (int)std::min<int64_t>(MLP_SPLITS, (n + 127) / 128); }

static int64_t mlp_dz_plan(const MlpDims& D, int64_t n, MlpDz& Z) {
  Z.np = (n + 63) / 64 * 64;
  int64_t at = 0;
  for (int l = 0; l < D.nlayer; ++l) {
    Z.off[l] = at;
    at += D.N[l] * Z.np;
  }
  return at;
}

int64_t mlp_dz_floats(const MlpDims& D, int64_t n) {
  MlpDz Z;
  return mlp_dz_plan(D, n, Z);
}

template <int HT>
static void dz_launch(const MlpDims& D, const MlpDz& Z, const uint16_t* P, const float* cache, const float* dy,
                      int64_t n, float* dzT, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_dz<HT>, dim3((unsigned)(Z.np / 64)), dim3(256), 0, s, D, Z, P, cache, dy, n, dzT);
}

// dzT: mlp_dz_floats(D, n) floats; part: mlp_splits(n) x nparam floats.
void mlp_backward(const MlpDims& D, const uint16_t* P, const float* cache, const float* dy, int64_t n, float* grad,
                  float* dzT, float* part, hipStream_t s) {
  MlpDz Z;
  mlp_dz_plan(D, n, Z);
  switch (D.d_hidden / 16) {
    case 1: dz_launch<1>(D, Z, P, cache, dy, n, dzT, s); break;
    case 2: dz_launch<2>(D, Z, P, cache, dy, n, dzT, s); break;
    case 3: dz_launch<3>(D, Z, P, cache, dy, n, dzT, s); break;
    case 4: dz_launch<4>(D, Z, P, cache, dy, n, dzT, s); break;
    case 5: dz_launch<5>(D, Z, P, cache, dy, n, dzT, s); break;
    case 6: dz_launch<6>(D, Z, P, cache, dy, n, dzT, s); break;
    case 7: dz_launch<7>(D, Z, P, cache, dy, n, dzT, s); break;
    default: dz_launch<8>(D, Z, P, cache, dy, n, dzT, s);
  }
  const int splits = mlp_splits(n);
  const int64_t chunk = ((Z.np + splits - 1) / splits + 15) / 16 * 16;
  int tiles = 0;
  for (int l = 0; l < D.nlayer; ++l) tiles += mlp_dw_tiles(D.N[l], D.K[l]);
  hipLaunchKernelGGL(k_mlp_dw, dim3(tiles, splits), dim3(64), 0, s, D, Z, dzT, cache, n, chunk, part);
  hipLaunchKernelGGL(k_mlp_dw_reduce, dim3(blocks_for(D.nparam, 256)), dim3(256), 0, s, part, splits, D.nparam, grad);
}

void mlp_adam(int64_t np, float* master, float* m, float* v, const float* g, uint16_t* pbf, float lr, float b1,
              float b2, float eps, int t, hipStream_t s) {
  const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
  hipLaunchKernelGGL(k_mlp_adam, dim3(blocks_for(np, 256)), dim3(256), 0, s, np, master, m, v, g, pbf, lr, b1, b2,
                     eps, c1, c2);
}

void mlp_to_bf16(int64_t np, const float* master, uint16_t* pbf, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_to_bf16, dim3(blocks_for(np, 256)), dim3(256), 0, s, np, master, pbf);
}

void mlp_features(const CellMap& M, int64_t ncells, const double* cond, float* x, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_features, dim3(blocks_for(ncells, 256)), dim3(256), 0, s, M, ncells, cond, x);
}

void mlp_targets(const CellMap& M, int64_t ncells, const double* q, const double* cond, double gamma, float* t,
                 hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_targets, dim3(blocks_for(ncells, 256)), dim3(256), 0, s, M, ncells, q, cond, gamma, t);
}

void mlp_to_state(const CellMap& M, int64_t ncells, const float* y, const double* cond, double gamma, double* q,
                  hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_to_state, dim3(blocks_for(ncells, 256)), dim3(256), 0, s, M, ncells, y, cond, gamma, q);
}

}  // namespace cfd
