// Surrogate network for ln k_s: an ensemble of MLPs 6 -> 128 -> 128 -> 128 -> 1
// (SiLU), trained and queried with the kernels below.
//
// Numerics, two precisions chosen per model: FP32 master weights always.
//  - BF16: BF16 copies of the weights (round to nearest even) feed the
//    forward pass; the two 128x128 layers run on v_mfma_f32_16x16x16_bf16
//    (BF16 inputs, FP32 accumulation); hidden activations are rounded to
//    BF16 before entering the next layer.
//  - FP32: the master weights and FP32 activations throughout; the 128x128
//    layers run on v_mfma_f32_16x16x4_f32.
// In both the 6-wide input layer and the 128-wide output dot run in FP32.  Inputs are the six
// physical quantities (LET, b, V, gap, dose per pulse, pulse rate),
// standardised as (log x - mu) / sigma.  Optionally the network learns the
// residual of ln k_s over an analytic baseline, -ln f_Jaffe - ln f_Boag:
// Jaffe's collection efficiency of a track parallel to the field (eq.
// Jaffe_noangle, with the averaged D and mu) times Boag's ln(1+u)/u for the
// uniform dose; the baseline is evaluated here in FP64.  The output is the
// standardised residual.  Training: mean squared error over each minibatch,
// backward in FP32 (with BF16 the casts pass gradients straight through),
// Adam.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "internal.h"
#include "reduce.h"

namespace it {
namespace {

constexpr int kH = 128, kIn = 6;
constexpr int oW1 = 0, ob1 = oW1 + kH * kIn, oW2 = ob1 + kH, ob2 = oW2 + kH * kH, oW3 = ob2 + kH,
              ob3 = oW3 + kH * kH, ow4 = ob3 + kH, ob4 = ow4 + kH, kP = ob4 + 1;  // 34049
constexpr int kPpad = (kP + 63) / 64 * 64;
constexpr int kTileS = 64;       // samples per query tile, and per BF16 forward tile
constexpr int64_t kFewQueries = 8192;
constexpr int kActStride = kH + 4;  // padded BF16 row (avoids LDS bank conflicts)

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int kGL = 32;  // Gauss-Legendre nodes of the Jaffe integral

struct Header {
  int32_t members, step;
  float mu[kIn], sigma[kIn], lo[kIn], hi[kIn];
  float t_mu, t_sigma;
  int32_t use_baseline;
  int32_t precision;  // IT_MLP_BF16 or IT_MLP_FP32
  // averaged diffusion and mobility, alpha, W [eV], mu+ + mu-, ion pairs
  // per cm^3 and mGy
  double D, mu_avg, alpha, W, mu_sum, pairs_per_mGy;
  double gl_x[kGL], gl_w[kGL];  // nodes and weights on [-1, 1]
};

struct Model {  // device pointers carved from the model buffer
  Header* hdr;
  float* master;      // [M][kP]
  float* m;           // [M][kP]
  float* v;           // [M][kP]
  unsigned short* w;  // [M][kPpad] BF16
};

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

size_t model_bytes(int M) {
  return align256(sizeof(Header)) + 3 * align256((size_t)M * kP * sizeof(float)) +
         align256((size_t)M * kPpad * sizeof(unsigned short));
}

Model carve_model(void* base, int M) {
  char* p = (char*)base;
  Model md;
  md.hdr = (Header*)p;
  p += align256(sizeof(Header));
  md.master = (float*)p;
  p += align256((size_t)M * kP * sizeof(float));
  md.m = (float*)p;
  p += align256((size_t)M * kP * sizeof(float));
  md.v = (float*)p;
  p += align256((size_t)M * kP * sizeof(float));
  md.w = (unsigned short*)p;
  return md;
}

// The BF16 weights of a model of M members (for kernels that learn M from the
// header).
__device__ inline const unsigned short* bf16_weights(const Model& md, int M) {
  const size_t field = ((size_t)M * kP * sizeof(float) + 255) / 256 * 256;
  return (const unsigned short*)((const char*)md.master + 3 * field);
}

struct TrainWs {  // per member: [M][n][...]
  float *z, *a1, *a2, *a3, *h1, *h2, *h3, *y, *dy, *d1, *d2, *d3, *grad, *loss, *base;
};

size_t train_ws_bytes(int M, int64_t n) {
  const size_t nh = (size_t)M * n * kH * sizeof(float);
  return 9 * align256(nh) + align256((size_t)M * n * kIn * 4) + 2 * align256((size_t)M * n * 4) +
         align256((size_t)M * kP * 4) + align256((size_t)M * 4) + align256((size_t)n * 4);
}

TrainWs carve_train(void* base, int M, int64_t n) {
  char* p = (char*)base;
  auto take = [&](size_t bytes) {
    float* r = (float*)p;
    p += align256(bytes);
    return r;
  };
  const size_t nh = (size_t)M * n * kH * sizeof(float);
  TrainWs w;
  w.a1 = take(nh);
  w.a2 = take(nh);
  w.a3 = take(nh);
  w.h1 = take(nh);
  w.h2 = take(nh);
  w.h3 = take(nh);
  w.d1 = take(nh);
  w.d2 = take(nh);
  w.d3 = take(nh);
  w.z = take((size_t)M * n * kIn * 4);
  w.y = take((size_t)M * n * 4);
  w.dy = take((size_t)M * n * 4);
  w.grad = take((size_t)M * kP * 4);
  w.loss = take((size_t)M * 4);
  w.base = take((size_t)n * 4);
  return w;
}

// Analytic baseline of ln k_s for one query (FP64): -ln f_J - ln f_B with
// f_J = (y1/y2) e^{-y1} [Ei(y1 + ln(1+y2)) - Ei(y1)], written as
// (y1/y2) int_0^{ln(1 + ln(1+y2)/y1)} exp(y1 (e^w - 1)) dw (no overflow for
// large y1), y1 = 8 pi D/(alpha N0), y2 = 2 d D/(mu b^2 E), N0 = LET/W, and
// f_B = ln(1+u)/u with u = alpha/(mu+ + mu-) n0 d^2/V.  The quadrature is
// summed in four parts of kGL/4 nodes (added in order).
struct BaseArgs {
  double y1, y2, upper;
};

__device__ inline BaseArgs base_args(const Header& H, const float* x) {
  const double let = x[0], b = x[1], V = x[2], d = x[3];
  const double E = V / d;
  const double N0 = let * 1.0e7 / H.W;
  BaseArgs a;
  a.y1 = 8.0 * M_PI * H.D / (H.alpha * N0);
  a.y2 = 2.0 * d * H.D / (H.mu_avg * b * b * E);
  a.upper = log1p(log1p(a.y2) / a.y1);
  return a;
}

constexpr int kBaseParts = 4, kPartLen = kGL / kBaseParts;

// Value of the integrand at node q.
__device__ inline double base_node(const Header& H, const BaseArgs& a, int q) {
  const double w = 0.5 * a.upper * (H.gl_x[q] + 1.0);
  return exp(a.y1 * expm1(w));
}

// Part `part` of the weighted sum.
__device__ inline double base_part(const Header& H, const BaseArgs& a, int part) {
  double s = 0.0;
  for (int q = part * kPartLen; q < (part + 1) * kPartLen; ++q) s = fma(H.gl_w[q], base_node(H, a, q), s);
  return s;
}

__device__ inline double base_finish(const Header& H, const float* x, const BaseArgs& a, double sum) {
  const double V = x[2], d = x[3], dose = x[4];
  const double fJ = a.y1 / a.y2 * (sum * 0.5 * a.upper);
  const double u = H.alpha / H.mu_sum * dose * H.pairs_per_mGy * d * d / V;
  const double fB = u > 0.0 ? log1p(u) / u : 1.0;
  return -log(fJ) - log(fB);
}

__device__ double baseline(const Header& H, const float* x) {
  const BaseArgs a = base_args(H, x);
  double s = base_part(H, a, 0);
  for (int p = 1; p < kBaseParts; ++p) s += base_part(H, a, p);
  return base_finish(H, x, a, s);
}

// Baseline of the S samples of a tile: the block's 256 threads share the
// quadratures (an exponential of FP64 takes as long as dozens of the network's
// instructions).  Thread p S + s takes the p-th share of the nodes of sample
// s0 + s into v[.][s]: the sum of a part where four threads share a sample,
// the integrand's values where more do.  After a barrier thread s < S calls
// base_of, which adds its sample's sums.  Either way they are the sums of
// baseline(), term by term, so that a sample's baseline does not depend on
// the tile it is in.
template <int S>
constexpr int kBaseRows = 256 / S == kBaseParts ? kBaseParts : kGL;

template <int S>
__device__ inline void base_parts(const Header& H, const float* __restrict__ X, int64_t n, int64_t s0,
                                  double (*v)[S]) {
  constexpr int kShare = kGL * S / 256;  // nodes of a thread
  const int p = threadIdx.x / S, s = threadIdx.x % S;
  const int64_t gs = s0 + s;
  if (!H.use_baseline || gs >= n) return;
  const BaseArgs a = base_args(H, X + gs * kIn);
  if constexpr (kBaseRows<S> == kBaseParts) {
    v[p][s] = base_part(H, a, p);
  } else {
    for (int q = p * kShare; q < (p + 1) * kShare; ++q) v[q][s] = base_node(H, a, q);
  }
}

template <int S>
__device__ inline double base_of(const Header& H, const float* __restrict__ X, int64_t gs, const double (*v)[S],
                                 int s) {
  if (!H.use_baseline) return 0.0;
  const float* x = X + gs * kIn;
  double part[kBaseParts];
  if constexpr (kBaseRows<S> == kBaseParts) {
    for (int p = 0; p < kBaseParts; ++p) part[p] = v[p][s];
  } else {
    for (int p = 0; p < kBaseParts; ++p) part[p] = 0.0;
    for (int q = 0; q < kPartLen; ++q)
      for (int p = 0; p < kBaseParts; ++p) {
        const int node = p * kPartLen + q;
        part[p] = fma(H.gl_w[node], v[node][s], part[p]);
      }
  }
  double sum = part[0];
  for (int p = 1; p < kBaseParts; ++p) sum += part[p];
  return base_finish(H, x, base_args(H, x), sum);
}

__device__ inline unsigned short to_bf16(float f) {  // round to nearest even
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ inline float from_bf16(unsigned short h) { return __uint_as_float((unsigned)h << 16); }
// The logistic function 1/(1 + e^-a) from the hardware base-2 exponential
// (e^-a = 2^(-a log2 e)) and reciprocal: a few instructions instead of a
// full-precision exponential and division, about 1e-6 relative for the
// pre-activations the network sees (the rounding of -a log2 e dominates).
// Large |a| saturate correctly: 2^(+big) = inf gives 0, 2^(-big) = 0 gives 1.
__device__ inline float logistic(float a) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-a * 1.44269504088896341f));
}
__device__ inline float silu(float a) { return a * logistic(a); }
__device__ inline float dsilu(float a) {
  const float s = logistic(a);
  return s * (1.0f + a * (1.0f - s));
}

struct ForwardOut {  // optional stores of the training forward (member slices)
  float *z, *a1, *a2, *a3, *h1, *h2, *h3, *y;
};

// ---------------------------------------------------------------------------
// FP32 models.  A block of 256 threads takes a tile of S samples of one
// member; wave w computes units 32 w .. 32 w + 31 of every sample of the tile,
// so each wave reads its own part of a layer's weights, straight from the L2
// into registers one layer ahead, and only the activations go through LDS.
// Products run on v_mfma_f32_16x16x4f32 (A[i][k]: lane i + 16 k, B[k][j]: lane
// j + 16 k, D[i][j]: lane j + 16 (i/4), item i % 4).  Which four of the 128
// terms a product takes is free as long as A and B agree: product e takes
// terms 32 q + e, q = lane / 16, so that a lane's terms are consecutive in
// memory and in LDS (16-byte loads).  Column j of output tile t is unit
// 32 w + 2 j + t, so a thread's two units of a sample are neighbours.  Every
// per-element value a thread computes sits at (sample 16 st + 4 (lane/16) + v,
// unit 32 w + 2 (lane % 16) + t) in every layer, so the pre-activations stay in
// its registers for the backward pass.
//
// What bounds it: the FP32 matrix instructions (32 cycles each) where the
// tiles fill the chip (half of their peak with 65 536 queries: 219 us, 233 with
// the weights staged in LDS), the latency of a tile's chain of layers where
// they do not (100 queries 32 us, 68 in tiles of 64; 2048 samples of four
// members, a training tile per CU, 28 us, 51 with 64 samples on half of the
// CUs).
typedef float float4u_t __attribute__((ext_vector_type(4), aligned(4)));  // parameters are not aligned further
typedef float float2u_t __attribute__((ext_vector_type(2), aligned(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));

// A wave's part of a 128 x 128 layer: term 32 q + e of tiles t = 0, 1.
struct WFrag {
  float v[2][32];
};

// Forward: B[k][j] = W[unit][k].
__device__ inline void wload_fwd(WFrag& f, const float* __restrict__ W) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const float* row = W + (32 * wave + 2 * (lane & 15) + t) * kH + 32 * (lane >> 4);
#pragma unroll
    for (int e = 0; e < 32; e += 4) {
      const float4u_t x = *(const float4u_t*)(row + e);
#pragma unroll
      for (int c = 0; c < 4; ++c) f.v[t][e + c] = x[c];
    }
  }
}

// Backward: B[k][j] = W[k][unit].
__device__ inline void wload_bwd(WFrag& f, const float* __restrict__ W) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const float* col = W + 32 * (lane >> 4) * kH + 32 * wave + 2 * (lane & 15);
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    const float2u_t x = *(const float2u_t*)(col + e * kH);
    f.v[0][e] = x[0];
    f.v[1][e] = x[1];
  }
}

// acc[st][t]: the products of the activations of S samples with the wave's
// weights.
template <int S>
__device__ inline void mm_f32(const float (*in)[kActStride], const WFrag& f, float4_t (&acc)[S / 16][2]) {
  const int lane = threadIdx.x % 64;
#pragma unroll
  for (int st = 0; st < S / 16; ++st)
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[st][t] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int e = 0; e < 32; e += 4) {
    float4_t a[S / 16];
#pragma unroll
    for (int st = 0; st < S / 16; ++st) a[st] = *(const float4_t*)&in[16 * st + (lane & 15)][32 * (lane >> 4) + e];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int st = 0; st < S / 16; ++st)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          acc[st][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[st][c], f.v[t][e + c], acc[st][t], 0, 0, 0);
  }
}

// Calls f(st, v, s) for the samples s of the tile that this thread's values
// belong to.
template <int S, class F>
__device__ inline void each_sample(F f) {
  const int lane = threadIdx.x % 64;
#pragma unroll
  for (int st = 0; st < S / 16; ++st)
#pragma unroll
    for (int v = 0; v < 4; ++v) f(st, v, 16 * st + 4 * (lane >> 4) + v);
}

// The first unit of this thread (the second is the next).
__device__ inline int unit0() { return 32 * (int)(threadIdx.x / 64) + 2 * (int)(threadIdx.x & 15); }

// Standardised inputs of the tile.
template <int S>
__device__ inline void inputs_f32(const Header& H, const float* __restrict__ X, int64_t n, int64_t s0, float* zs) {
  for (int q = threadIdx.x; q < S * kIn; q += 256) {
    const int64_t gs = s0 + q / kIn;
    const int i = q % kIn;
    zs[q] = gs < n ? (logf(X[gs * kIn + i]) - H.mu[i]) / H.sigma[i] : 0.0f;
  }
}

// A thread's parameters outside the 128 x 128 matrices.
struct SmallP {
  float w1[2][kIn], b1[2], b2[2], b3[2];
};

__device__ inline void sload(const float* __restrict__ master, SmallP& sp) {
  const int o = unit0();
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int i = 0; i < kIn; ++i) sp.w1[t][i] = master[oW1 + (o + t) * kIn + i];
    sp.b1[t] = master[ob1 + o + t];
    sp.b2[t] = master[ob2 + o + t];
    sp.b3[t] = master[ob3 + o + t];
  }
}

// Pre-activation of the first layer of sample s, unit t.
__device__ inline float first_layer(const SmallP& sp, const float* zs, int s, int t) {
  float a = sp.b1[t];
#pragma unroll
  for (int i = 0; i < kIn; ++i) a += sp.w1[t][i] * zs[s * kIn + i];
  return a;
}

// Output layer: four partial dot products of 32 terms per sample, into
// yp[p][s]; w4 (128 values, then b4) in LDS.  The sum is output_f32's.
template <int S>
__device__ inline void dots_f32(const float (*act)[kActStride], const float* w4, float (*yp)[S]) {
  const int s = threadIdx.x % S, p = threadIdx.x / S;
  if (p < 4) {
    float y = 0.0f;
#pragma unroll 8
    for (int i = 32 * p; i < 32 * p + 32; ++i) y += w4[i] * act[s][i];
    yp[p][s] = y;
  }
}

template <int S>
__device__ inline float output_f32(const float* w4, const float (*yp)[S], int s) {
  return w4[kH] + (((yp[0][s] + yp[1][s]) + yp[2][s]) + yp[3][s]);
}

// One FP32 training step's per-sample work for a tile of samples of one
// member: the forward pass, the loss gradient dy = 2 (y - t_std) / n, and the
// pre-activation gradients of the three hidden layers; activations and
// gradients go out for the weight gradients.  The baseline of each sample is
// written by the member-0 blocks (the loss kernel reads it).  Tiles of 32
// samples: a minibatch of 2048 of four members then puts a block on every CU.
constexpr int kTrainS = 32;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void train_tile_f32_kernel(
    Model md, const float* __restrict__ X, const float* __restrict__ t_, int64_t n, TrainWs ws) {
  constexpr int S = kTrainS, NS = S / 16;
  __shared__ float zs[S * kIn];
  __shared__ __align__(16) float act[2][S][kActStride];
  __shared__ float w4[kH + 1];
  __shared__ float yp[4][S];
  __shared__ float dys[S];
  __shared__ double bp[kBaseRows<S>][S];
  const Header& H = *md.hdr;
  const int tid = threadIdx.x;
  const int m = blockIdx.y;
  const int64_t s0 = (int64_t)blockIdx.x * S;
  const float* master = md.master + (size_t)m * kP;
  const size_t nh = (size_t)n * kH;
  const int o = unit0();
  WFrag fa, fb;
  SmallP sp;
  wload_fwd(fa, master + oW2);
  sload(master, sp);
  if (tid < kH + 1) w4[tid] = master[ow4 + tid];
  inputs_f32<S>(H, X, n, s0, zs);
  // the baseline and target of each sample, while W2 is on its way
  base_parts<S>(H, X, n, s0, bp);
  __syncthreads();
  const int64_t gt = s0 + tid;
  float ty = 0.0f;
  if (tid < S && gt < n) {
    const float base = (float)base_of<S>(H, X, gt, bp, tid);
    if (m == 0) ws.base[gt] = base;
    ty = (t_[gt] - base - H.t_mu) / H.t_sigma;
  }
  if (tid < S * kIn && s0 + tid / kIn < n) ws.z[(size_t)m * n * kIn + s0 * kIn + tid] = zs[tid];
  // a pair of values of sample s: into LDS and, for real samples, to memory
  auto put = [&](float (*to)[kActStride], float* mem, int s, float x, float y) {
    if (to) *(float2_t*)&to[s][o] = float2_t{x, y};
    if (s0 + s < n) *(float2_t*)(mem + (size_t)m * nh + (s0 + s) * kH + o) = float2_t{x, y};
  };
  float a1[NS][4][2], a2[NS][4][2], a3[NS][4][2];
  each_sample<S>([&](int st, int v, int s) {
#pragma unroll
    for (int t = 0; t < 2; ++t) a1[st][v][t] = first_layer(sp, zs, s, t);
    put(act[0], ws.h1, s, silu(a1[st][v][0]), silu(a1[st][v][1]));
  });
  __syncthreads();
  float4_t acc[NS][2];
  wload_fwd(fb, master + oW3);
  mm_f32<S>(act[0], fa, acc);
  each_sample<S>([&](int st, int v, int s) {
#pragma unroll
    for (int t = 0; t < 2; ++t) a2[st][v][t] = acc[st][t][v] + sp.b2[t];
    put(act[1], ws.h2, s, silu(a2[st][v][0]), silu(a2[st][v][1]));
  });
  __syncthreads();
  wload_bwd(fa, master + oW3);
  mm_f32<S>(act[1], fb, acc);
  each_sample<S>([&](int st, int v, int s) {
#pragma unroll
    for (int t = 0; t < 2; ++t) a3[st][v][t] = acc[st][t][v] + sp.b3[t];
    put(act[0], ws.h3, s, silu(a3[st][v][0]), silu(a3[st][v][1]));
  });
  __syncthreads();
  wload_bwd(fb, master + oW2);
  dots_f32<S>(act[0], w4, yp);
  __syncthreads();
  if (tid < S) {
    float dy = 0.0f;
    if (gt < n) {
      const float y = output_f32<S>(w4, yp, tid);
      ws.y[(size_t)m * n + gt] = y;
      dy = 2.0f * (y - ty) / (float)n;
      ws.dy[(size_t)m * n + gt] = dy;
    }
    dys[tid] = dy;
  }
  __syncthreads();
  // d3 = dy w4 silu'(a3), then back through the layers: d = (d W) silu'(a)
  each_sample<S>([&](int st, int v, int s) {
    put(act[1], ws.d3, s, dys[s] * w4[o] * dsilu(a3[st][v][0]), dys[s] * w4[o + 1] * dsilu(a3[st][v][1]));
  });
  __syncthreads();
  mm_f32<S>(act[1], fa, acc);
  each_sample<S>([&](int st, int v, int s) {
    put(act[0], ws.d2, s, acc[st][0][v] * dsilu(a2[st][v][0]), acc[st][1][v] * dsilu(a2[st][v][1]));
  });
  __syncthreads();
  mm_f32<S>(act[0], fb, acc);
  each_sample<S>([&](int st, int v, int s) {
    put(nullptr, ws.d1, s, acc[st][0][v] * dsilu(a1[st][v][0]), acc[st][1][v] * dsilu(a1[st][v][1]));
  });
}

// ---------------------------------------------------------------------------
// BF16 models: hidden activations rounded to BF16 before the next layer,
// the 128 x 128 layers on v_mfma_f32_16x16x16_bf16.
//
// Forward pass of one member over samples [s0, s0 + 64) (256 threads).
// Leaves the standardised outputs in ys[64] (LDS).
template <bool STORE>
__device__ void forward_tile_bf16(const Header& H, const float* __restrict__ master,
                                  const unsigned short* __restrict__ w, const float* __restrict__ X, int64_t n,
                                  int64_t s0, float* zs /*[64][6]*/, unsigned short (*act)[kTileS][kActStride],
                                  float* ys, const ForwardOut& st) {
  const int tid = threadIdx.x;
  const int wave = tid / 64, lane = tid % 64;
  // standardised inputs
  for (int q = tid; q < kTileS * kIn; q += 256) {
    const int s = q / kIn, i = q % kIn;
    const int64_t gs = s0 + s;
    float zv = 0.0f;
    if (gs < n) zv = (logf(X[gs * kIn + i]) - H.mu[i]) / H.sigma[i];
    zs[q] = zv;
    if (STORE && gs < n) st.z[gs * kIn + i] = zv;
  }
  __syncthreads();
  // layer 1 (FP32 arithmetic on the BF16 weights)
  for (int q = tid; q < kTileS * kH; q += 256) {
    const int s = q / kH, o = q % kH;
    float a = master[ob1 + o];
#pragma unroll
    for (int i = 0; i < kIn; ++i) a += from_bf16(w[oW1 + o * kIn + i]) * zs[s * kIn + i];
    const unsigned short h = to_bf16(silu(a));
    act[0][s][o] = h;
    const int64_t gs = s0 + s;
    if (STORE && gs < n) {
      st.a1[gs * kH + o] = a;
      st.h1[gs * kH + o] = from_bf16(h);
    }
  }
  __syncthreads();
  // layers 2 and 3: wave w owns samples 16w..16w+15
#pragma unroll
  for (int layer = 0; layer < 2; ++layer) {
    const int oW = layer == 0 ? oW2 : oW3, ob = layer == 0 ? ob2 : ob3;
    const unsigned short (*in)[kActStride] = act[layer];
    unsigned short (*out)[kActStride] = act[1 - layer];
    float* sa = layer == 0 ? st.a2 : st.a3;
    float* sh = layer == 0 ? st.h2 : st.h3;
    const int arow = wave * 16 + (lane & 15);  // A: sample row of this lane
    const int kq = 4 * (lane >> 4);            // A/B: k offset within the 16-wide step
#pragma unroll 1
    for (int nt = 0; nt < kH / 16; ++nt) {
      float4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
      const int bo = nt * 16 + (lane & 15);  // B: output column of this lane
#pragma unroll
      for (int kk = 0; kk < kH / 16; ++kk) {
        const int k = kk * 16 + kq;
        short4_t a, b;
        a[0] = (short)in[arow][k];
        a[1] = (short)in[arow][k + 1];
        a[2] = (short)in[arow][k + 2];
        a[3] = (short)in[arow][k + 3];
        const unsigned short* wr = w + oW + bo * kH + k;
        b[0] = (short)wr[0];
        b[1] = (short)wr[1];
        b[2] = (short)wr[2];
        b[3] = (short)wr[3];
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
      }
      // D[i][j]: sample i = 4 (lane/16) + v, output j = lane % 16
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int s = wave * 16 + 4 * (lane >> 4) + v;
        const float a = acc[v] + master[ob + bo];
        const unsigned short h = to_bf16(silu(a));
        out[s][bo] = h;
        const int64_t gs = s0 + s;
        if (STORE && gs < n) {
          sa[gs * kH + bo] = a;
          sh[gs * kH + bo] = from_bf16(h);
        }
      }
    }
    __syncthreads();
  }
  // output layer (FP32 dot); act[0] holds h3
  if (tid < kTileS) {
    float y = master[ob4];
    for (int i = 0; i < kH; ++i) y += from_bf16(w[ow4 + i]) * from_bf16(act[0][tid][i]);
    ys[tid] = y;
    const int64_t gs = s0 + tid;
    if (STORE && gs < n) st.y[gs] = y;
  }
  __syncthreads();
}

__global__ __launch_bounds__(256) void forward_train_bf16_kernel(Model md, const float* X, int64_t n, TrainWs ws) {
  if (blockIdx.y == 0 && threadIdx.x < kTileS) {  // baseline of each sample (member independent)
    const int64_t gs = (int64_t)blockIdx.x * kTileS + threadIdx.x;
    if (gs < n) ws.base[gs] = md.hdr->use_baseline ? (float)baseline(*md.hdr, X + gs * kIn) : 0.0f;
  }
  __shared__ float zs[kTileS * kIn];
  __shared__ unsigned short act[2][kTileS][kActStride];
  __shared__ float ys[kTileS];
  const int m = blockIdx.y;
  const size_t nh = (size_t)n * kH;
  ForwardOut st{ws.z + (size_t)m * n * kIn, ws.a1 + m * nh, ws.a2 + m * nh, ws.a3 + m * nh,
                ws.h1 + m * nh, ws.h2 + m * nh, ws.h3 + m * nh, ws.y + (size_t)m * n};
  forward_tile_bf16<true>(*md.hdr, md.master + (size_t)m * kP, md.w + (size_t)m * kPpad, X, n,
                          (int64_t)blockIdx.x * kTileS, zs, act, ys, st);
}

// Per-sample deltas of a BF16 model: dy = 2 (y - t)/n, then the
// pre-activation gradients of the three hidden layers (block of 128
// threads = hidden units; the casts pass gradients straight through).
__global__ __launch_bounds__(128) void delta_bf16_kernel(Model md, const float* t, int64_t n, TrainWs ws) {
  __shared__ float d[kH];
  const int m = blockIdx.y, o = threadIdx.x;
  const int64_t s = blockIdx.x;
  const size_t nh = (size_t)n * kH, row = m * nh + (size_t)s * kH;
  const unsigned short* w = md.w + (size_t)m * kPpad;
  const float ty = (t[s] - ws.base[s] - md.hdr->t_mu) / md.hdr->t_sigma;
  const float dy = 2.0f * (ws.y[(size_t)m * n + s] - ty) / (float)n;
  if (o == 0) ws.dy[(size_t)m * n + s] = dy;
  float da = dy * from_bf16(w[ow4 + o]) * dsilu(ws.a3[row + o]);
  ws.d3[row + o] = da;
  d[o] = da;
  __syncthreads();
  float g = 0.0f;
  for (int j = 0; j < kH; ++j) g += from_bf16(w[oW3 + j * kH + o]) * d[j];
  da = g * dsilu(ws.a2[row + o]);
  ws.d2[row + o] = da;
  __syncthreads();
  d[o] = da;
  __syncthreads();
  g = 0.0f;
  for (int j = 0; j < kH; ++j) g += from_bf16(w[oW2 + j * kH + o]) * d[j];
  ws.d1[row + o] = g * dsilu(ws.a1[row + o]);
}

// ---------------------------------------------------------------------------
// Weight gradients G[o][i] = sum_s delta[s][o] * in[s][i] on FP32 MFMA
// (v_mfma_f32_16x16x4f32, four samples each).  Slice
// z takes the samples 16 g + 4 z .. 16 g + 4 z + 3, g = 0, 1, ..., in order, and
// the four slices' sums are added, in order, where they are used (adam_kernel,
// sum_grad_kernel): deterministic.  Blocks x < 16 each a 64 x 32 part of a
// 128 x 128 layer's matrix (a wave 32 outputs by 16 inputs, two tiles that share
// B; row r of output tile a is unit 2 r + a), blocks 16..18 W1 and b1, b2,
// b3, and blocks 19..21 w4 and b4, a 16 x 16 tile per wave.  One 16 x 16 tile of all samples per block, as
// before, read every activation eight times: 29 us for 2048 samples of four
// members; 17 us now.
constexpr int kSlices = 4, kMatrixBlocks = 16, kLastBlock = kMatrixBlocks + 3, kGradBlocks = kLastBlock + 3;

struct GradSums {  // [slices][members] sums of a slice, strides in floats
  float* p;
  int slices;  // kSlices, or 1: a block adds the slices itself
  size_t slice_stride, member_stride;
};

// One operand of the products: this lane's element of the sample rows behind
// `rows` (row_floats each), `at` bytes into the first of them (kNone: zero),
// plus a constant.  Rows are taken as buffers, so that a load costs no address
// arithmetic and 32 groups of samples are in flight (with 64-bit addresses the
// compiler kept three: 38 us).
struct Operand {
  const float* rows;
  int row_floats;
  unsigned at;
  float plus;
};

constexpr unsigned kNone = 0xfffffff0u;  // an offset outside every buffer
constexpr int kU = 32;                   // groups of four samples in flight
constexpr int kTail = 8;                 // the same of a slice's last groups
constexpr int kFew = 16;                 // the same where a block adds the slices itself

template <class V>
__device__ inline void load_rows(const Operand& o, int64_t s, int group, bool there, V& v) {
  const uint64_t a = (uint64_t)(o.rows + s * o.row_floats);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  const unsigned bytes = 16u * kU * o.row_floats * 4u;
  const __amdgpu_buffer_rsrc_t r =
      __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), 0, bytes, 0x00027000);
  const unsigned at = there ? o.at : kNone;
  if constexpr (sizeof(V) == 8) v = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, at, group * 16 * o.row_floats, 0));
  else v = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(r, at, group * 16 * o.row_floats, 0));
}

// One slice of the samples: acc[a] += A x B, the A operand one or two tiles.
template <int NA>
__device__ inline void slice_sum(const Operand& A, const Operand& B, int64_t n, int z, float4_t (&acc)[NA]) {
  typedef float a_t __attribute__((ext_vector_type(NA)));
  const int k = (threadIdx.x % 64) >> 4;
#pragma unroll
  for (int a = 0; a < NA; ++a) acc[a] = {0.0f, 0.0f, 0.0f, 0.0f};
  int64_t s = 4 * z;
  for (; s + 16 * (kU - 1) + 3 < n; s += 16 * kU) {
    a_t x[kU];
    float y[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      load_rows(A, s, 4 * u, true, x[u]);
      load_rows(B, s, 4 * u, true, y[u]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int a = 0; a < NA; ++a)
        acc[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][a], y[u] + B.plus, acc[a], 0, 0, 0);
  }
  // the rest, kTail groups in flight, missing samples as zeros
  for (; s < n; s += 16 * kTail) {
    a_t x[kTail];
    float y[kTail];
#pragma unroll
    for (int u = 0; u < kTail; ++u) {
      const bool there = s + 16 * u + k < n;
      load_rows(A, s, 4 * u, there, x[u]);
      load_rows(B, s, 4 * u, there, y[u]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kTail; ++u) {
      if (s + 16 * u >= n) break;  // uniform
      const float plus = s + 16 * u + k < n ? B.plus : 0.0f;
#pragma unroll
      for (int a = 0; a < NA; ++a)
        acc[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][a], y[u] + plus, acc[a], 0, 0, 0);
    }
  }
}

// All slices of few samples, added in order.  Group g of four samples belongs to
// slice g % kSlices: the loads of all slices go out together, and the kernel is
// short (a launch starts by fetching its code; with slice_sum's four times over,
// 64 samples took 6.2 us, 1.4 more than without slices).
template <int NA>
__device__ inline void all_slices(const Operand& A, const Operand& B, int64_t n, float4_t (&sum)[NA]) {
  typedef float a_t __attribute__((ext_vector_type(NA)));
  const int k = (threadIdx.x % 64) >> 4;
  float4_t acc[kSlices][NA];
#pragma unroll
  for (int z = 0; z < kSlices; ++z)
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[z][a] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
  for (int64_t s = 0; s < n; s += 4 * kFew) {
    a_t x[kFew];
    float y[kFew];
#pragma unroll
    for (int u = 0; u < kFew; ++u) {
      const bool there = s + 4 * u + k < n;
      load_rows(A, s, u, there, x[u]);
      load_rows(B, s, u, there, y[u]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kFew; ++u) {
      if (s + 4 * u >= n) break;  // uniform
      const float plus = s + 4 * u + k < n ? B.plus : 0.0f;
#pragma unroll
      for (int a = 0; a < NA; ++a)
        acc[u % kSlices][a] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][a], y[u] + plus, acc[u % kSlices][a], 0, 0, 0);
    }
  }
#pragma unroll
  for (int a = 0; a < NA; ++a) sum[a] = acc[0][a];
#pragma unroll
  for (int z = 1; z < kSlices; ++z)
#pragma unroll
    for (int a = 0; a < NA; ++a) sum[a] += acc[z][a];
}

// The block's slice (SLICES = kSlices), or all of them.
template <int SLICES, int NA>
__device__ inline void block_sum(const Operand& A, const Operand& B, int64_t n, int z, float4_t (&sum)[NA]) {
  if constexpr (SLICES == kSlices) slice_sum(A, B, n, z, sum);
  else all_slices(A, B, n, sum);
}

// All blocks of a member and slice run on one XCD (the dispatcher deals blocks
// to the 8 XCDs in turn), so that each L2 reads its own part of the activations
// once, not every L2 all of them.
template <int SLICES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void wgrad_kernel(TrainWs ws, int64_t n,
                                                                                             int members,
                                                                                             GradSums sums) {
  const int pair = blockIdx.x % 8 + 8 * (blockIdx.x / (8 * kGradBlocks));
  if (pair >= members * SLICES) return;
  const int m = pair / SLICES, z = pair % SLICES;
  float* out = sums.p + z * sums.slice_stride + m * sums.member_stride;
  const size_t nh = (size_t)n * kH;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int r = lane & 15, k = lane >> 4;
  const int x = blockIdx.x / 8 % kGradBlocks;
  // element e of row k (the sample of the group that this lane loads)
  auto in_row = [&](int row_floats, int e) { return (unsigned)(k * row_floats + e) * 4u; };
  if (x < kMatrixBlocks) {
    const int layer = x / 8, part = x % 8;  // 0: W2, 1: W3
    const int o0 = 64 * (part & 1) + 32 * (wave & 1), i0 = 32 * (part >> 1) + 16 * (wave >> 1);
    const Operand A{(layer ? ws.d3 : ws.d2) + m * nh, kH, in_row(kH, o0 + 2 * r), 0.0f};
    const Operand B{(layer ? ws.h2 : ws.h1) + m * nh, kH, in_row(kH, i0 + r), 0.0f};
    float4_t acc[2];
    block_sum<SLICES>(A, B, n, z, acc);
    float* w = out + (layer ? oW3 : oW2);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int v = 0; v < 4; ++v) w[(o0 + 2 * (4 * k + v) + a) * kH + i0 + r] = acc[a][v];  // D[4 k + v][r]
    return;
  }
  if (x >= kLastBlock) {  // w4 and b4: row 0 of A is dy; B 16 units of h3, or ones
    const int tile = 4 * (x - kLastBlock) + wave;
    if (tile > kH / 16) return;
    const bool ones = tile == kH / 16;
    const Operand A{ws.dy + (size_t)m * n, 1, r == 0 ? in_row(1, 0) : kNone, 0.0f};
    const Operand B{ws.h3 + m * nh, kH, ones ? kNone : in_row(kH, 16 * tile + r), ones ? 1.0f : 0.0f};
    float4_t acc[1];
    block_sum<SLICES>(A, B, n, z, acc);
    if (k == 0) {  // D[0][r]
      if (!ones) out[ow4 + 16 * tile + r] = acc[0][0];
      else if (r == 0) out[ob4] = acc[0][0];
    }
    return;
  }
  // columns of B: the inputs (first layer only), then ones
  const int layer = x - kMatrixBlocks, nin = layer == 0 ? kIn : 0;
  const Operand A{(layer == 0 ? ws.d1 : layer == 1 ? ws.d2 : ws.d3) + m * nh, kH, in_row(kH, 32 * wave + 2 * r), 0.0f};
  const Operand B{ws.z + (size_t)m * n * kIn, kIn, r < nin ? in_row(kIn, r) : kNone, r == nin ? 1.0f : 0.0f};
  float4_t acc[2];
  block_sum<SLICES>(A, B, n, z, acc);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int o = 32 * wave + 2 * (4 * k + v) + a;
      if (r < nin) out[oW1 + o * kIn + r] = acc[a][v];
      if (r == nin) out[(layer == 0 ? ob1 : layer == 1 ? ob2 : ob3) + o] = acc[a][v];
    }
}

__device__ inline float summed_grad(const GradSums& sums, int m, int k) {
  const float* p = sums.p + m * sums.member_stride + k;
  float g = p[0];
  for (int z = 1; z < sums.slices; ++z) g += p[z * sums.slice_stride];
  return g;
}

__global__ void sum_grad_kernel(GradSums sums, int M, float* grad) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < (int64_t)M * kP) grad[q] = summed_grad(sums, (int)(q / kP), (int)(q % kP));
}

__global__ void adam_kernel(Model md, GradSums sums, int M, float lr, int step) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)M * kP) return;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float g = summed_grad(sums, (int)(q / kP), (int)(q % kP));
  const float m = b1 * md.m[q] + (1.0f - b1) * g;
  const float v = b2 * md.v[q] + (1.0f - b2) * g * g;
  md.m[q] = m;
  md.v[q] = v;
  const float mh = m / (1.0f - powf(b1, (float)step));
  const float vh = v / (1.0f - powf(b2, (float)step));
  const float p = md.master[q] - lr * mh / (sqrtf(vh) + eps);
  md.master[q] = p;
  const int64_t mem = q / kP, k = q % kP;
  md.w[mem * kPpad + k] = to_bf16(p);
}

__global__ void to_bf16_kernel(Model md, int M) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)M * kP) return;
  md.w[(q / kP) * kPpad + q % kP] = to_bf16(md.master[q]);
}

__global__ __launch_bounds__(1024) void loss_kernel(Model md, const float* t, int64_t n, TrainWs ws) {
  const int m = blockIdx.x;
  __shared__ float part[16];
  float s = 0.0f;
  for (int64_t q = threadIdx.x; q < n; q += 1024) {
    const float r = ws.y[(size_t)m * n + q] - (t[q] - ws.base[q] - md.hdr->t_mu) / md.hdr->t_sigma;
    s += r * r;
  }
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
  if (threadIdx.x % 64 == 0) part[threadIdx.x / 64] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float tot = 0.0f;
    for (int w = 0; w < 16; ++w) tot += part[w];
    ws.loss[m] = tot / (float)n;
  }
}

// Ensemble query: mean and spread (max - min) of ln k_s over the members,
// out-of-box test of the standardised inputs, fallback flag and the number
// of flagged queries per block.  Per tile of 64 queries, after the members'
// forward passes (LDS ys, summed into ysum/ymin/ymax).
template <int S>
__device__ inline void query_finish(const Header& H, const float* __restrict__ X, int64_t n, int64_t s0,
                                    float spread_tol, const float* zs, float* ysum, float* ymin, float* ymax,
                                    double (*bp)[S], float* mean, float* spread, unsigned char* fallback,
                                    int* cnt, int* block_count) {
  const int tid = threadIdx.x;
  base_parts<S>(H, X, n, s0, bp);
  __syncthreads();
  if (tid < S && s0 + tid < n) {
    const int64_t gs = s0 + tid;
    const float base = (float)base_of<S>(H, X, gs, bp, tid);
    ysum[tid] += (float)H.members * base;
    ymin[tid] += base;
    ymax[tid] += base;
    bool out = false;
    for (int i = 0; i < kIn; ++i) {
      const float z = zs[tid * kIn + i];
      out = out || !(z >= H.lo[i] && z <= H.hi[i]);
    }
    const float sp = ymax[tid] - ymin[tid];
    mean[gs] = ysum[tid] / (float)H.members;
    spread[gs] = sp;
    const bool fb = out || !(sp <= spread_tol);
    fallback[gs] = fb ? 1 : 0;
    if (fb) atomicAdd(cnt, 1);
  }
  __syncthreads();
  if (tid == 0 && block_count) block_count[blockIdx.x] = *cnt;
}

template <int S>
__device__ inline void query_accumulate(const Header& H, int m, const float* ys, float* ysum, float* ymin,
                                        float* ymax) {
  const int tid = threadIdx.x;
  if (tid < S) {
    const float v = ys[tid] * H.t_sigma + H.t_mu;
    ysum[tid] = m == 0 ? v : ysum[tid] + v;
    ymin[tid] = m == 0 ? v : fminf(ymin[tid], v);
    ymax[tid] = m == 0 ? v : fmaxf(ymax[tid], v);
  }
  __syncthreads();
}

// Tiles of S queries; the members in turn, each one's weights on their way
// while the one before is computed.  64 queries per tile where that fills the
// chip (two blocks per CU); 16 for few queries, which are then spread over
// four times the CUs and whose chain of layers is four times shorter.
template <int S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void query_f32_kernel(
    Model md, const float* __restrict__ X, int64_t n, float spread_tol, float* mean, float* spread,
    unsigned char* fallback, int* block_count) {
  constexpr int NH = S >= 32 ? 2 : 1, HS = S / NH;  // halves of the tile
  __shared__ float zs[S * kIn];
  __shared__ __align__(16) float act[S][kActStride];
  __shared__ float w4[kH + 1];
  __shared__ float yp[4][S];
  __shared__ float ys[S], ymin[S], ymax[S], ysum[S];
  __shared__ double bp[kBaseRows<S>][S];
  __shared__ int cnt;
  const Header& H = *md.hdr;
  if (H.precision != IT_MLP_FP32) return;
  const int64_t s0 = (int64_t)blockIdx.x * S;
  const int tid = threadIdx.x, o = unit0();
  const int members = H.members;
  if (tid == 0) cnt = 0;
  WFrag fa, fb;
  SmallP sp;
  wload_fwd(fa, md.master + oW2);
  sload(md.master, sp);
  inputs_f32<S>(H, X, n, s0, zs);
  __syncthreads();
  for (int m = 0; m < members; ++m) {
    const float* master = md.master + (size_t)m * kP;
    if (tid < kH + 1) w4[tid] = master[ow4 + tid];  // its last readers passed a barrier
    float4_t acc[2][HS / 16][2];
    // the first layer of half h, and the activations of its last product
    auto first = [&](int h) {
      each_sample<HS>([&](int, int, int s) {
        const int hs = h * HS + s;
        *(float2_t*)&act[hs][o] = float2_t{silu(first_layer(sp, zs, hs, 0)), silu(first_layer(sp, zs, hs, 1))};
      });
    };
    auto activate = [&](int h, const float (&b)[2]) {
      each_sample<HS>([&](int st, int v, int s) {
        *(float2_t*)&act[h * HS + s][o] =
            float2_t{silu(acc[h][st][0][v] + b[0]), silu(acc[h][st][1][v] + b[1])};
      });
    };
    // One half's products and the other half's activations side by side.
    first(0);
    __syncthreads();
    wload_fwd(fb, master + oW3);
    mm_f32<HS>(act, fa, acc[0]);
    if (NH == 2) first(NH - 1);
    __syncthreads();
    if (NH == 2) mm_f32<HS>(act + HS, fa, acc[NH - 1]);
    activate(0, sp.b2);
    __syncthreads();
    if (m + 1 < members) wload_fwd(fa, master + kP + oW2);
    mm_f32<HS>(act, fb, acc[0]);
    if (NH == 2) activate(NH - 1, sp.b2);
    __syncthreads();
    if (NH == 2) mm_f32<HS>(act + HS, fb, acc[NH - 1]);
    activate(0, sp.b3);
    if (NH == 2) {
      __syncthreads();
      activate(NH - 1, sp.b3);
    }
    if (m + 1 < members) sload(master + kP, sp);
    __syncthreads();
    dots_f32<S>(act, w4, yp);
    __syncthreads();
    if (tid < S) ys[tid] = output_f32<S>(w4, yp, tid);
    query_accumulate<S>(H, m, ys, ysum, ymin, ymax);
  }
  query_finish<S>(H, X, n, s0, spread_tol, zs, ysum, ymin, ymax, bp, mean, spread, fallback, &cnt, block_count);
}

__global__ __launch_bounds__(256) void query_bf16_kernel(Model md, const float* __restrict__ X, int64_t n,
                                                         float spread_tol, float* mean, float* spread,
                                                         unsigned char* fallback, int* block_count) {
  __shared__ float zs[kTileS * kIn];
  __shared__ unsigned short act[2][kTileS][kActStride];
  __shared__ float ys[kTileS], ymin[kTileS], ymax[kTileS], ysum[kTileS];
  __shared__ double bp[kBaseRows<kTileS>][kTileS];
  __shared__ int cnt;
  const Header& H = *md.hdr;
  if (H.precision != IT_MLP_BF16) return;
  const unsigned short* weights = bf16_weights(md, H.members);
  const int64_t s0 = (int64_t)blockIdx.x * kTileS;
  if (threadIdx.x == 0) cnt = 0;
  const ForwardOut none{};
  for (int m = 0; m < H.members; ++m) {
    forward_tile_bf16<false>(H, md.master + (size_t)m * kP, weights + (size_t)m * kPpad, X, n, s0, zs, act, ys,
                             none);
    query_accumulate<kTileS>(H, m, ys, ysum, ymin, ymax);
  }
  query_finish<kTileS>(H, X, n, s0, spread_tol, zs, ysum, ymin, ymax, bp, mean, spread, fallback, &cnt, block_count);
}
// Ordered compaction of the flagged query indices: an exclusive scan of the
// per-block counts (one block), then each block writes its flagged indices
// in order.
__global__ __launch_bounds__(1024) void scan_kernel(const int* block_count, int nblocks, int* block_off,
                                                    int64_t* total) {
  __shared__ int buf[1024];
  int carry = 0;
  for (int b0 = 0; b0 < nblocks; b0 += 1024) {
    const int b = b0 + threadIdx.x;
    const int v = b < nblocks ? block_count[b] : 0;
    buf[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {  // inclusive Hillis-Steele scan
      const int u = threadIdx.x >= off ? buf[threadIdx.x - off] : 0;
      __syncthreads();
      buf[threadIdx.x] += u;
      __syncthreads();
    }
    if (b < nblocks) block_off[b] = carry + buf[threadIdx.x] - v;
    const int last = buf[1023];
    __syncthreads();
    carry += last;
  }
  if (threadIdx.x == 0) *total = carry;
}

// As many flagged queries as lie before tile b, the sum of the tiles' counts
// in front of it: with few tiles cheaper than a scan in a launch of its own.
constexpr int kScanTiles = 4096;  // tiles from which the scan is one

// off: the scan's offsets, or null: summed here (and the total written by the
// last block).
__global__ __launch_bounds__(kTileS) void scatter_kernel(const unsigned char* fallback, int64_t n,
                                                         const int* block_count, const int* off, int64_t* total,
                                                         int64_t* idx) {
  const int64_t s0 = (int64_t)blockIdx.x * kTileS;
  const int64_t gs = s0 + threadIdx.x;
  const bool f = gs < n && fallback[gs];
  const unsigned long long mask = __ballot(f);
  int first;
  if (off) {
    first = off[blockIdx.x];
  } else {
    int v = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kTileS) v += block_count[b];
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    first = v;
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = first + __popcll(mask);
  }
  if (f && idx) {
    const unsigned long long below = mask & ((1ull << threadIdx.x) - 1ull);
    idx[first + __popcll(below)] = gs;
  }
}

// The same for few queries, from their flags, by one block.
__global__ __launch_bounds__(1024) void compact_kernel(const unsigned char* fallback, int64_t n, int64_t* total,
                                                       int64_t* idx) {
  __shared__ int count[16];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  int first = 0;
  for (int64_t s0 = 0; s0 < n; s0 += 1024) {
    const int64_t gs = s0 + threadIdx.x;
    const bool f = gs < n && fallback[gs];
    const unsigned long long mask = __ballot(f);
    if (lane == 0) count[wave] = __popcll(mask);
    __syncthreads();
    int before = first;
    for (int w = 0; w < 16; ++w) {
      if (w < wave) before += count[w];
      first += count[w];
    }
    if (f && idx) idx[before + __popcll(mask & ((1ull << lane) - 1ull))] = gs;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = first;
}

__global__ void baseline_kernel(Model md, const float* X, int64_t n, double* out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) out[q] = baseline(*md.hdr, X + q * kIn);
}

// Gauss-Legendre nodes and weights on [-1, 1] by Newton iteration on the
// Legendre polynomial (three-term recursion).
void gauss_legendre(int n, double* x, double* w) {
  for (int i = 0; i < n; ++i) {
    double z = std::cos(M_PI * (i + 0.75) / (n + 0.5));
    double dp = 0.0;
    for (int it = 0; it < 100; ++it) {
      double p0 = 1.0, p1 = z;
      for (int k = 2; k <= n; ++k) {
        const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      dp = n * (z * p1 - p0) / (z * z - 1.0);
      const double dz = p1 / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-16) break;
    }
    x[i] = z;
    w[i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
}

}  // namespace
}  // namespace it

using namespace it;

extern "C" {

int it_mlp_model_bytes(int32_t members, size_t* bytes) {
  if (!bytes || members < 1 || members > 64) return IT_EINVAL;
  *bytes = model_bytes(members);
  return IT_OK;
}

int it_mlp_init(void* d_model, int32_t members, const float* h_params, const float* h_norm, const double* h_phys,
                int32_t precision, void* stream_) {
  clear_stale_error();
  if (!d_model || !h_params || !h_norm || members < 1 || members > 64) return IT_EINVAL;
  if (precision != IT_MLP_BF16 && precision != IT_MLP_FP32) return IT_EINVAL;
  hipStream_t s = (hipStream_t)stream_;
  Model md = carve_model(d_model, members);
  Header h;
  std::memset(&h, 0, sizeof(h));
  h.members = members;
  h.precision = precision;
  for (int i = 0; i < kIn; ++i) {
    h.mu[i] = h_norm[i];
    h.sigma[i] = h_norm[kIn + i];
    h.lo[i] = h_norm[2 * kIn + i];
    h.hi[i] = h_norm[3 * kIn + i];
    if (!(h.sigma[i] > 0.0f) || !(h.lo[i] <= h.hi[i])) return IT_EINVAL;
  }
  h.t_mu = h_norm[4 * kIn];
  h.t_sigma = h_norm[4 * kIn + 1];
  if (!(h.t_sigma > 0.0f)) return IT_EINVAL;
  if (h_phys) {
    h.use_baseline = 1;
    h.D = h_phys[0];
    h.mu_avg = h_phys[1];
    h.alpha = h_phys[2];
    h.W = h_phys[3];
    h.mu_sum = h_phys[4];
    h.pairs_per_mGy = h_phys[5];
    for (int q = 0; q < 6; ++q)
      if (!(std::isfinite(h_phys[q]) && h_phys[q] > 0.0)) return IT_EINVAL;
    gauss_legendre(kGL, h.gl_x, h.gl_w);
  }
  if (hipMemcpyAsync(md.hdr, &h, sizeof(h), hipMemcpyHostToDevice, s) != hipSuccess ||
      hipMemcpyAsync(md.master, h_params, (size_t)members * kP * 4, hipMemcpyHostToDevice, s) != hipSuccess ||
      hipMemsetAsync(md.m, 0, (size_t)members * kP * 4, s) != hipSuccess ||
      hipMemsetAsync(md.v, 0, (size_t)members * kP * 4, s) != hipSuccess)
    return IT_EHIP;
  hipLaunchKernelGGL(to_bf16_kernel, dim3((members * kP + 255) / 256), dim3(256), 0, s, md, members);
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return IT_EHIP;
  return IT_OK;
}

int it_mlp_train_ws_bytes(int32_t members, int64_t n, size_t* bytes) {
  if (!bytes || members < 1 || members > 64 || n < 1) return IT_EINVAL;
  *bytes = train_ws_bytes(members, n);
  return IT_OK;
}

// The slices' sums go where the pre-activations stood, which nothing reads any
// more then; with few samples that is too small, and few blocks do: each then
// adds the slices itself, into the gradient's place.
static GradSums grad_sums(const TrainWs& w, int M, int64_t n) {
  if ((size_t)n * 3 * kH >= (size_t)kSlices * kPpad) return GradSums{w.a1, kSlices, (size_t)M * kPpad, (size_t)kPpad};
  return GradSums{w.grad, 1, 0, (size_t)kP};
}

static int launch_grad(const Model& md, int M, bool f32, const float* X, const float* t, int64_t n,
                       const TrainWs& w, const GradSums& sums, hipStream_t s) {
  if (f32) {
    const int nb = (int)((n + kTrainS - 1) / kTrainS);
    hipLaunchKernelGGL(train_tile_f32_kernel, dim3(nb, M), dim3(256), 0, s, md, X, t, n, w);
  } else {
    const int nb = (int)((n + kTileS - 1) / kTileS);
    hipLaunchKernelGGL(forward_train_bf16_kernel, dim3(nb, M), dim3(256), 0, s, md, X, n, w);
    hipLaunchKernelGGL(delta_bf16_kernel, dim3((unsigned)n, M), dim3(kH), 0, s, md, t, n, w);
  }
  const dim3 grid((M * sums.slices + 7) / 8 * 8 * kGradBlocks);
  if (sums.slices == kSlices) hipLaunchKernelGGL(wgrad_kernel<kSlices>, grid, dim3(256), 0, s, w, n, M, sums);
  else hipLaunchKernelGGL(wgrad_kernel<1>, grid, dim3(256), 0, s, w, n, M, sums);
  return hipGetLastError() == hipSuccess ? IT_OK : IT_EHIP;
}

int it_mlp_grad(const void* d_model, int32_t members, const float* d_X, const float* d_t, int64_t n,
                float* d_grad, float* h_loss, void* d_ws, size_t ws_bytes, void* stream_) {
  clear_stale_error();
  if (!d_model || !d_X || !d_t || !d_grad || n < 1 || members < 1 || members > 64) return IT_EINVAL;
  if (!d_ws || ws_bytes < train_ws_bytes(members, n)) return IT_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream_;
  Model md = carve_model((void*)d_model, members);
  TrainWs w = carve_train(d_ws, members, n);
  Header h;
  if (hipMemcpyAsync(&h, md.hdr, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return IT_EHIP;
  const GradSums sums = grad_sums(w, members, n);
  int rc = launch_grad(md, members, h.precision == IT_MLP_FP32, d_X, d_t, n, w, sums, s);
  if (rc) return rc;
  hipLaunchKernelGGL(sum_grad_kernel, dim3((members * kP + 255) / 256), dim3(256), 0, s, sums, members, d_grad);
  if (h_loss) {
    hipLaunchKernelGGL(loss_kernel, dim3(members), dim3(1024), 0, s, md, d_t, n, w);
    if (hipMemcpyAsync(h_loss, w.loss, members * 4, hipMemcpyDeviceToHost, s) != hipSuccess) return IT_EHIP;
  }
  return hipStreamSynchronize(s) == hipSuccess ? IT_OK : IT_EHIP;
}

int it_mlp_train(void* d_model, int32_t members, const float* d_X, const float* d_t, int64_t n, int64_t batch,
                 int32_t steps, float lr, float lr_final, int32_t log_every, float* h_loss, void* d_ws,
                 size_t ws_bytes, void* stream_) {
  clear_stale_error();
  if (!d_model || !d_X || !d_t || n < 1 || steps < 0 || members < 1 || members > 64 || !(lr > 0.0f) ||
      !(lr_final > 0.0f) || batch < 0 || batch > n)
    return IT_EINVAL;
  const int64_t rows = batch ? batch : n;
  if (n % rows) return IT_EINVAL;  // the minibatches tile the data
  if (!d_ws || ws_bytes < train_ws_bytes(members, rows)) return IT_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream_;
  Model md = carve_model(d_model, members);
  TrainWs w = carve_train(d_ws, members, rows);
  Header h;
  if (hipMemcpyAsync(&h, md.hdr, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return IT_EHIP;
  const int64_t nbatch = n / rows;
  const GradSums sums = grad_sums(w, members, rows);
  int nlog = 0;
  for (int k = 0; k < steps; ++k) {
    // minibatch: the next contiguous window of the data, continuing across calls
    const int64_t b0 = ((h.step + k) % nbatch) * rows;
    const float* X = d_X + b0 * kIn;
    const float* t = d_t + b0;
    int rc = launch_grad(md, members, h.precision == IT_MLP_FP32, X, t, rows, w, sums, s);
    if (rc) return rc;
    if (h_loss && log_every > 0 && k % log_every == 0) {
      hipLaunchKernelGGL(loss_kernel, dim3(members), dim3(1024), 0, s, md, t, rows, w);
      if (hipMemcpyAsync(h_loss + (size_t)nlog * members, w.loss, members * 4, hipMemcpyDeviceToHost, s) !=
          hipSuccess)
        return IT_EHIP;
      ++nlog;
    }
    // cosine decay from lr to lr_final over the steps of this call
    const double frac = steps > 1 ? (double)k / (double)(steps - 1) : 0.0;
    const double lr0 = lr, lr1 = lr_final;  // in FP64: the end points are exact
    const float lr_k = (float)(lr1 + 0.5 * (lr0 - lr1) * (1.0 + std::cos(M_PI * frac)));
    hipLaunchKernelGGL(adam_kernel, dim3((members * kP + 255) / 256), dim3(256), 0, s, md, sums, members, lr_k,
                       h.step + k + 1);
    if (hipGetLastError() != hipSuccess) return IT_EHIP;
  }
  h.step += steps;
  if (hipMemcpyAsync(md.hdr, &h, sizeof(h), hipMemcpyHostToDevice, s) != hipSuccess) return IT_EHIP;
  return hipStreamSynchronize(s) == hipSuccess ? IT_OK : IT_EHIP;
}

int it_mlp_baseline(const void* d_model, const float* d_X, int64_t n, double* d_out, void* stream_) {
  clear_stale_error();
  if (!d_model || n < 0 || (n > 0 && (!d_X || !d_out))) return IT_EINVAL;
  if (n == 0) return IT_OK;
  hipStream_t s = (hipStream_t)stream_;
  Model md = carve_model((void*)d_model, 1);  // only the header is read
  hipLaunchKernelGGL(baseline_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, md, d_X, n, d_out);
  return hipGetLastError() == hipSuccess ? IT_OK : IT_EHIP;
}

int it_mlp_query_ws_bytes(int64_t nq, size_t* bytes) {
  if (!bytes || nq < 0) return IT_EINVAL;
  const int64_t nb = (nq + kTileS - 1) / kTileS;
  *bytes = align256((size_t)nb * 4) * 2 + 256;
  return IT_OK;
}

}  // extern "C"

namespace it {
namespace {

// The query with its scratch (per-tile fallback counts and offsets, the
// total) at d_ws, it_mlp_query_ws_bytes(nq) bytes.
int query(const void* d_model, const float* d_X, int64_t nq, float spread_tol, float* d_mean, float* d_spread,
          unsigned char* d_fallback, int64_t* d_fallback_idx, int64_t* h_nfallback, void* d_ws, hipStream_t s) {
  if (nq == 0) {
    if (h_nfallback) *h_nfallback = 0;
    return IT_OK;
  }
  const Model md = carve_model((void*)d_model, 1);  // header and master weights; the kernels read the members
  const int nb = (int)((nq + kTileS - 1) / kTileS);
  char* p = (char*)d_ws;
  int* counts = (int*)p;
  int* offs = (int*)(p + align256((size_t)nb * 4));
  int64_t* total = (int64_t*)(p + 2 * align256((size_t)nb * 4));
  // The model's precision stands in its header: both kernels are launched, and
  // the other one's blocks end at once (reading the header back first took a
  // copy and a synchronisation, 20 us).  Few queries go in tiles of 16 and are
  // compacted by one block: 8192 of them are still two blocks per CU.
  const bool few = nq <= kFewQueries;
  if (few)
    hipLaunchKernelGGL(query_f32_kernel<16>, dim3((unsigned)((nq + 15) / 16)), dim3(256), 0, s, md, d_X, nq, spread_tol,
                       d_mean, d_spread, d_fallback, (int*)nullptr);
  else
    hipLaunchKernelGGL(query_f32_kernel<kTileS>, dim3(nb), dim3(256), 0, s, md, d_X, nq, spread_tol, d_mean, d_spread,
                       d_fallback, counts);
  hipLaunchKernelGGL(query_bf16_kernel, dim3(nb), dim3(256), 0, s, md, d_X, nq, spread_tol, d_mean, d_spread,
                     d_fallback, counts);
  if (few) {
    hipLaunchKernelGGL(compact_kernel, dim3(1), dim3(1024), 0, s, d_fallback, nq, total, d_fallback_idx);
  } else {
    const bool scan = nb > kScanTiles;
    if (scan) hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, s, counts, nb, offs, total);
    if (!scan || d_fallback_idx)
      hipLaunchKernelGGL(scatter_kernel, dim3(nb), dim3(kTileS), 0, s, d_fallback, nq, counts, scan ? offs : nullptr,
                         total, d_fallback_idx);
  }
  if (hipGetLastError() != hipSuccess) return IT_EHIP;
  if (h_nfallback) {
    if (hipMemcpyAsync(h_nfallback, total, 8, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return IT_EHIP;
  }
  return IT_OK;
}

// Scratch of the allocation-free query: a file-scope device array, one copy
// per GPU, held until the process ends.  Its device address is taken once
// per device (with that device current) and kept: in host code the array's
// name is only a stand-in for it.  Nothing in it needs to start at zero
// (every query tile writes its own count, the scan writes the offsets and
// the total).
constexpr int64_t kStaticQueries = IT_MLP_QUERY_STATIC_MAX;
constexpr size_t kStaticScratchBytes = 2 * (((size_t)kStaticQueries / kTileS * 4 + 255) / 256 * 256) + 256;
__device__ __align__(256) char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_ptr[kMaxDevices] = {};

void* static_scratch() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
    scratch_ptr[dev] = ptr;
  }
  return scratch_ptr[dev];
}

}  // namespace
}  // namespace it

extern "C" {

int it_mlp_query(const void* d_model, const float* d_X, int64_t nq, float spread_tol, float* d_mean,
                 float* d_spread, unsigned char* d_fallback, int64_t* d_fallback_idx, int64_t* h_nfallback,
                 void* d_ws, size_t ws_bytes, void* stream_) {
  clear_stale_error();
  if (!d_model || nq < 0 || (nq > 0 && (!d_X || !d_mean || !d_spread || !d_fallback))) return IT_EINVAL;
  size_t need;
  it_mlp_query_ws_bytes(nq, &need);
  if (!d_ws || ws_bytes < need) return IT_EWORKSPACE;
  return query(d_model, d_X, nq, spread_tol, d_mean, d_spread, d_fallback, d_fallback_idx, h_nfallback, d_ws,
               (hipStream_t)stream_);
}

int it_mlp_query_static(const void* d_model, const float* d_X, int64_t nq, float spread_tol, float* d_mean,
                        float* d_spread, unsigned char* d_fallback, int64_t* d_fallback_idx, int64_t* h_nfallback,
                        void* stream_) {
  clear_stale_error();
  if (!d_model || nq < 0 || nq > kStaticQueries || (nq > 0 && (!d_X || !d_mean || !d_spread || !d_fallback)))
    return IT_EINVAL;
  size_t need;
  it_mlp_query_ws_bytes(nq, &need);
  if (need > kStaticScratchBytes) return IT_EINVAL;
  void* ws = static_scratch();
  if (!ws) return IT_EHIP;
  return query(d_model, d_X, nq, spread_tol, d_mean, d_spread, d_fallback, d_fallback_idx, h_nfallback, ws,
               (hipStream_t)stream_);
}

}  // extern "C"
