// MLP cost model: the learned selector that stands in for the decision tree
// (section 5.1 of the paper compares an MLP with its decision trees; here
// the network regresses each chosen kernel's relative performance and the
// selection is the argmax).
//
// Network 6 -> 64 -> 64 -> k, ReLU after both hidden layers, linear output,
// y = x W^T + b with W row-major [out][in].  Features of a problem:
//   [log2 M / 12, log2 N / 12, log2 K / 12, log2 batch / 6, transA, transB]
// Targets: relative performance (Q16 / 65535) of the chosen kernels.  Loss:
// mean squared error over rows x k.  Full-batch Adam with bias correction.
//
// GPU layout: work-groups of 64 rows x one eighth of the gradients run forward
// and backward and write partial gradients per 32 rows; a second kernel sums
// the partials in block order (deterministic) and applies Adam.  A training
// run replays a captured hipGraph of several steps.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
#include <immintrin.h>
#endif

#include "kt_internal.hpp"

namespace kt {

static constexpr int MLP_IN = 6;
static constexpr int MLP_H = 64;
static constexpr int MLP_ROWS = 32;      // rows per partial gradient
static constexpr int MLP_MAX_K = 64;

struct MlpLayout {
  int k;
  int oW1, ob1, oW2, ob2, oW3, ob3, total;
  __host__ __device__ explicit MlpLayout(int kk) : k(kk) {
    oW1 = 0;
    ob1 = oW1 + MLP_H * MLP_IN;
    oW2 = ob1 + MLP_H;
    ob2 = oW2 + MLP_H * MLP_H;
    oW3 = ob2 + MLP_H;
    ob3 = oW3 + kk * MLP_H;
    total = ob3 + kk;
  }
};

// log2 of a positive integer, evaluated by the same float operations on the
// host and on the device so that host and device selection agree bit for bit
// (the math libraries' log2f may differ in the last place): v = m 2^e with
// e = floor(log2 v) and m in [1, 2] (float(v) scaled exactly by 2^-e), then
// log2 m = (2 / ln 2) atanh(t), t = (m - 1) / (m + 1) in [0, 1/3], from the
// odd series t (1 + t^2/3 + ... + t^14/15) (truncation below 5e-10), in
// Horner form with explicit fused multiply-adds.  Values <= 1 give 0.
__host__ __device__ inline float feature_log2(int64_t v) {
  if (v <= 1) return 0.f;
  const int e = 63 - __builtin_clzll((unsigned long long)v);
  const float m = ldexpf((float)v, -e);
  const float t = (m - 1.f) / (m + 1.f);
  const float t2 = t * t;
  float p = 1.f / 15.f;
  p = fmaf(p, t2, 1.f / 13.f);
  p = fmaf(p, t2, 1.f / 11.f);
  p = fmaf(p, t2, 1.f / 9.f);
  p = fmaf(p, t2, 1.f / 7.f);
  p = fmaf(p, t2, 1.f / 5.f);
  p = fmaf(p, t2, 1.f / 3.f);
  p = fmaf(p, t2, 1.f);
  const float u = 2.88539008f * t;   // 2 / ln 2
  return fmaf(u, p, (float)e);
}

__host__ __device__ inline void shape_features(const kt_shape& s, float* x) {
  x[0] = feature_log2(s.M) * (1.0f / 12.0f);
  x[1] = feature_log2(s.N) * (1.0f / 12.0f);
  x[2] = feature_log2(s.K) * (1.0f / 12.0f);
  x[3] = feature_log2(s.batch) * (1.0f / 6.0f);
  x[4] = (float)s.transA;
  x[5] = (float)s.transB;
}

// Features -> forward -> argmax (lowest index on ties): the position in the
// chosen list.  Shared by the batch selection kernel and the host launcher
// path, with the same operation order, so both pick the same kernel.
__host__ __device__ inline int mlp_forward_argmax(const kt_shape& shape, const float* P, int k) {
  const MlpLayout L(k);
  float x[MLP_IN], h1[MLP_H], h2[MLP_H];
  shape_features(shape, x);
  for (int o = 0; o < MLP_H; ++o) {
    float s = P[L.ob1 + o];
    for (int q = 0; q < MLP_IN; ++q) s = fmaf(x[q], P[L.oW1 + o * MLP_IN + q], s);
    h1[o] = fmaxf(s, 0.f);
  }
  for (int o = 0; o < MLP_H; ++o) {
    float s = P[L.ob2 + o];
    for (int q = 0; q < MLP_H; ++q) s = fmaf(h1[q], P[L.oW2 + o * MLP_H + q], s);
    h2[o] = fmaxf(s, 0.f);
  }
  int best = 0;
  float bv = 0.f;
  for (int o = 0; o < k; ++o) {
    float s = P[L.ob3 + o];
    for (int q = 0; q < MLP_H; ++q) s = fmaf(h2[q], P[L.oW3 + o * MLP_H + q], s);
    if (o == 0 || s > bv) { bv = s; best = o; }
  }
  return best;
}

__global__ void mlp_features_kernel(const kt_shape* __restrict__ shapes, int n, float* __restrict__ X) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) shape_features(shapes[i], X + (int64_t)i * MLP_IN);
}

// Targets: Y[i][j] = q[i][chosen[j]] / 65535 from the normalized table.
__global__ void mlp_targets_kernel(const uint16_t* __restrict__ Xq, int n, int d,
                                   const int32_t* __restrict__ chosen, int k, float* __restrict__ Y) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * k) return;
  const int64_t i = e / k;
  const int j = (int)(e % k);
  Y[e] = (float)Xq[i * d + chosen[j]] * (1.0f / 65535.0f);
}

// Forward and backward.  Writes one partial gradient (same layout as the
// parameters) and one partial sum of squared errors per block of MLP_ROWS
// rows; optionally the predictions.  step: the first work-group increments
// the Adam step counter.
//
// A work-group takes two blocks, one row per lane, and one of MLP_SLICES
// slices of the gradients: it runs the forward pass of its 64 rows (waves
// share the outputs of a layer and exchange them through LDS) and the backward
// pass down to its slice of the units.  In the products over units a weight is
// the same for every lane and comes by scalar loads; in the products over rows
// a lane is a unit, and the other factor, one value per row, is broadcast
// from a register lane by lane, so LDS carries one word per activation instead
// of two per multiply.  Every sum runs in the order r or i = 0, 1, ... of its
// block, one fused multiply-add each.  What bounds it is the chain of dependent
// phases of one step, not the chip: so sixteen waves, two per unit of the slice
// with one row block each.  3000 steps of 960 rows: 60 ms; eight waves that take
// both blocks 71; one work-group per block that read both factors of every
// multiply from LDS 113.
static constexpr int MLP_SLICES = 8;
static constexpr int MLP_WAVES = 16;
static constexpr int MLP_OUT_WAVES = 8;                // waves that share the last layer's outputs
static constexpr int MLP_GRAD_THREADS = MLP_WAVES * 64;
static constexpr int MLP_UNITS = MLP_H / MLP_WAVES;    // units of a layer per wave
static constexpr int MLP_LD = 65;                      // LDS row: 64 rows of the batch, odd stride
static_assert(2 * MLP_H / MLP_SLICES == MLP_WAVES, "one unit of a slice and one row block per wave");

__global__ void __launch_bounds__(MLP_GRAD_THREADS)
mlp_fwdbwd_kernel(const float* __restrict__ P, const float* __restrict__ X, const float* __restrict__ Y,
                  int n, int k, float* __restrict__ part, float* __restrict__ part_loss,
                  float* __restrict__ pred, int* __restrict__ step) {
  extern __shared__ float sm[];
  const MlpLayout L(k);
  float* Z1 = sm;                               // [unit][row], before the ReLU
  float* Z2 = Z1 + MLP_H * MLP_LD;
  float* D2 = Z2 + MLP_H * MLP_LD;              // dz2
  float* XS = D2 + MLP_H * MLP_LD;              // [row][6]
  float* DY = XS + 2 * MLP_ROWS * MLP_IN;       // [output][row]
  __shared__ float red[MLP_WAVES][2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = blockIdx.y;
  const int r0 = blockIdx.x * 2 * MLP_ROWS;
  const bool in = r0 + lane < n;
  if (blockIdx.x == 0 && slice == 0 && tid == 0 && step) *step += 1;

  // z1 = x W1^T + b1
  float x[MLP_IN];
#pragma unroll
  for (int i = 0; i < MLP_IN; ++i) x[i] = in ? X[(int64_t)(r0 + lane) * MLP_IN + i] : 0.f;
  if (wave == 0) {
#pragma unroll
    for (int i = 0; i < MLP_IN; ++i) XS[lane * MLP_IN + i] = x[i];
  }
  const int u0 = wave * MLP_UNITS;
#pragma unroll
  for (int q = 0; q < MLP_UNITS; ++q) {
    float s = P[L.ob1 + u0 + q];
#pragma unroll
    for (int i = 0; i < MLP_IN; ++i) s = fmaf(x[i], P[L.oW1 + (u0 + q) * MLP_IN + i], s);
    Z1[(u0 + q) * MLP_LD + lane] = s;
  }
  __syncthreads();
  float h[MLP_H];
  // z2 = relu(z1) W2^T + b2
#pragma unroll
  for (int i = 0; i < MLP_H; ++i) h[i] = fmaxf(Z1[i * MLP_LD + lane], 0.f);
#pragma unroll
  for (int q = 0; q < MLP_UNITS; ++q) {
    const float* w = P + L.oW2 + (u0 + q) * MLP_H;
    float s = P[L.ob2 + u0 + q];
#pragma unroll
    for (int i = 0; i < MLP_H; ++i) s = fmaf(h[i], w[i], s);
    Z2[(u0 + q) * MLP_LD + lane] = s;
  }
  __syncthreads();
  // y = relu(z2) W3^T + b3 ; dy = 2 (y - Y) / (n k) ; loss partial
#pragma unroll
  for (int i = 0; i < MLP_H; ++i) h[i] = fmaxf(Z2[i * MLP_LD + lane], 0.f);
  const float scale = 2.0f / ((float)n * (float)k);
  float lsum = 0.f;
  for (int o = wave; wave < MLP_OUT_WAVES && o < k; o += MLP_OUT_WAVES) {
    const float* w = P + L.oW3 + o * MLP_H;
    float s = P[L.ob3 + o];
#pragma unroll
    for (int i = 0; i < MLP_H; ++i) s = fmaf(h[i], w[i], s);
    float dy = 0.f;
    if (in) {
      if (pred && slice == 0) pred[(int64_t)(r0 + lane) * k + o] = s;
      if (Y) {
        const float diff = s - Y[(int64_t)(r0 + lane) * k + o];
        lsum = fmaf(diff, diff, lsum);
        dy = scale * diff;
      }
    }
    DY[o * MLP_LD + lane] = dy;
  }
  if (!part) return;   // inference only (uniform across the grid)
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o);   // within each block's 32 lanes
  if ((lane & 31) == 0) red[wave][lane >> 5] = lsum;
  __syncthreads();
  if (slice == 0 && tid < 2 && r0 + tid * MLP_ROWS < n) {
    float s = 0.f;
    for (int w = 0; w < MLP_OUT_WAVES; ++w) s += red[w][tid];
    part_loss[blockIdx.x * 2 + tid] = s;
  }
  // dz2 = (dy W3) * [z2 > 0]
  {
    float acc[MLP_UNITS];
#pragma unroll
    for (int q = 0; q < MLP_UNITS; ++q) acc[q] = 0.f;
    for (int o = 0; o < k; ++o) {
      const float dy = DY[o * MLP_LD + lane];
      const float* w = P + L.oW3 + o * MLP_H + u0;
#pragma unroll
      for (int q = 0; q < MLP_UNITS; ++q) acc[q] = fmaf(dy, w[q], acc[q]);
    }
#pragma unroll
    for (int q = 0; q < MLP_UNITS; ++q)
      D2[(u0 + q) * MLP_LD + lane] = Z2[(u0 + q) * MLP_LD + lane] > 0.f ? acc[q] : 0.f;
  }
  __syncthreads();
  // dz1 = (dz2 W2) * [z1 > 0], unit `unit` of this slice (both waves of a unit)
  const int unit = slice * (MLP_WAVES / 2) + wave / 2, half = wave % 2;
  float d1 = 0.f;
  {
    const float* w = P + L.oW2 + unit;
#pragma unroll 16
    for (int o = 0; o < MLP_H; ++o) d1 = fmaf(D2[o * MLP_LD + lane], w[o * MLP_H], d1);
    d1 = Z1[unit * MLP_LD + lane] > 0.f ? d1 : 0.f;
  }
  // lane r (and r + 32): row r of this wave's block
  const int mine = half * MLP_ROWS + lane % MLP_ROWS;
  const float d2 = D2[unit * MLP_LD + mine];
  d1 = __shfl(d1, mine);
  // products over the rows of one block: lane -> input unit, the factor of
  // row r broadcast from lane r
  auto lane_of = [](float v, int l) {
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), l));
  };
  if (r0 + half * MLP_ROWS >= n) return;
  float* g = part + (int64_t)(blockIdx.x * 2 + half) * L.total;
  // dW2[unit][i] = sum_r dz2[r][unit] relu(z1[r][i]);  db2
  float s = 0.f, sb = 0.f;
#pragma unroll
  for (int r = 0; r < MLP_ROWS; ++r) {
    const float v = lane_of(d2, r);
    s = fmaf(v, fmaxf(Z1[lane * MLP_LD + half * MLP_ROWS + r], 0.f), s);
    sb += v;
  }
  g[L.oW2 + unit * MLP_H + lane] = s;
  if (lane == 0) g[L.ob2 + unit] = sb;
  // dW1[unit][i] = sum_r dz1[r][unit] x[r][i];  db1
  s = 0.f;
  sb = 0.f;
  const int i6 = lane < MLP_IN ? lane : 0;
#pragma unroll
  for (int r = 0; r < MLP_ROWS; ++r) {
    const float v = lane_of(d1, r);
    s = fmaf(v, XS[(half * MLP_ROWS + r) * MLP_IN + i6], s);
    sb += v;
  }
  if (lane < MLP_IN) g[L.oW1 + unit * MLP_IN + lane] = s;
  if (lane == 0) g[L.ob1 + unit] = sb;
  // dW3[o][i] = sum_r dy[r][o] relu(z2[r][i]);  db3; output o on slice o % 8, waves of unit o / 8
  for (int o = wave / 2 * MLP_SLICES + slice; o < k; o += MLP_SLICES * MLP_WAVES / 2) {
    const float dy = DY[o * MLP_LD + mine];
    s = 0.f;
    sb = 0.f;
#pragma unroll
    for (int r = 0; r < MLP_ROWS; ++r) {
      const float v = lane_of(dy, r);
      s = fmaf(v, fmaxf(Z2[lane * MLP_LD + half * MLP_ROWS + r], 0.f), s);
      sb += v;
    }
    g[L.oW3 + o * MLP_H + lane] = s;
    if (lane == 0) g[L.ob3 + o] = sb;
  }
}

// Sum the block partials in block order; optionally write the gradient and
// loss, and optionally apply one Adam step (t read from *step).
__global__ void mlp_reduce_adam_kernel(float* __restrict__ P, const float* __restrict__ part,
                                       const float* __restrict__ part_loss, int nblocks, int total,
                                       float* __restrict__ grad_out, float* __restrict__ loss_out,
                                       float* __restrict__ m, float* __restrict__ v,
                                       const int* __restrict__ step, float lr, int adam) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e == 0 && loss_out) {
    float s = 0.f;
    for (int b = 0; b < nblocks; ++b) s += part_loss[b];
    *loss_out = s;   // sum of squared errors; the mean is this / (n k)
  }
  if (e >= total) return;
  float gsum = 0.f;
#pragma unroll 8
  for (int b = 0; b < nblocks; ++b) gsum += part[(int64_t)b * total + e];
  if (grad_out) grad_out[e] = gsum;
  if (adam) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const int t = *step;
    const float mm = b1 * m[e] + (1.f - b1) * gsum;
    const float vv = b2 * v[e] + (1.f - b2) * gsum * gsum;
    m[e] = mm;
    v[e] = vv;
    const float c1 = 1.f - powf(b1, (float)t);
    const float c2 = 1.f - powf(b2, (float)t);
    P[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  }
}

// Batch selection: features -> forward -> argmax (lowest index on ties) -> id.
__global__ void mlp_select_kernel(const kt_shape* __restrict__ shapes, int n, const float* __restrict__ P,
                                  int k, const int32_t* __restrict__ chosen, int32_t* __restrict__ ids) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  ids[i] = chosen[mlp_forward_argmax(shapes[i], P, k)];
}

static size_t a256(size_t v) { return (v + 255) & ~(size_t)255; }

struct MlpPlan {
  size_t oP, oM, oV, oG, oPart, oPL, oX, oY, oStep, oLoss, oShapes, oT, oQ, oChosen, total;
  int nblocks;
};

static MlpPlan mlp_plan(int n, int k, int d) {
  MlpPlan p;
  const MlpLayout L(k);
  p.nblocks = (n + MLP_ROWS - 1) / MLP_ROWS;
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o = a256(o + bytes); return at; };
  p.oP = take((size_t)L.total * 4);
  p.oM = take((size_t)L.total * 4);
  p.oV = take((size_t)L.total * 4);
  p.oG = take((size_t)L.total * 4);
  p.oPart = take((size_t)p.nblocks * L.total * 4);
  p.oPL = take((size_t)p.nblocks * 4);
  p.oX = take((size_t)n * MLP_IN * 4);
  p.oY = take((size_t)n * k * 4);
  p.oStep = take(4);
  p.oLoss = take(4);
  p.oShapes = take((size_t)n * sizeof(kt_shape));
  p.oT = take((size_t)n * d * 8);
  p.oQ = take((size_t)n * d * 2);
  p.oChosen = take((size_t)k * 4);
  p.total = o;
  return p;
}

static size_t fwdbwd_lds(int k) {
  return ((size_t)(3 * MLP_H + k) * MLP_LD + 2 * MLP_ROWS * MLP_IN) * 4;
}

static hipError_t launch_fwdbwd(const float* P, const float* X, const float* Y, int n, int k,
                                float* part, float* part_loss, float* pred, int* step, hipStream_t st) {
  const int nb = (n + MLP_ROWS - 1) / MLP_ROWS;
  hipLaunchKernelGGL(mlp_fwdbwd_kernel, dim3((nb + 1) / 2, part ? MLP_SLICES : 1),
                     dim3(MLP_GRAD_THREADS), fwdbwd_lds(k), st, P, X, Y, n, k, part, part_loss, pred,
                     step);
  return hipGetLastError();
}

static hipError_t set_lds_attr(int k) {
  return hipFuncSetAttribute((const void*)mlp_fwdbwd_kernel,
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)fwdbwd_lds(k));
}

// He-uniform initialisation U(+-sqrt(6 / fan_in)) from SplitMix64(seed),
// W1, W2, W3 in that order, row-major; zero biases.
static void he_uniform(std::vector<float>& P, int k, uint64_t seed) {
  const MlpLayout L(k);
  P.assign(L.total, 0.f);
  uint64_t state = seed;
  auto next_uniform = [&]() {
    uint64_t z = state + 0x9E3779B97F4A7C15ull;
    state = z;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (double)(z >> 11) * (1.0 / 9007199254740992.0);
  };
  auto fill = [&](int off, int fan_out, int fan_in) {
    const double bound = sqrt(6.0 / fan_in);
    for (int e = 0; e < fan_out * fan_in; ++e) P[off + e] = (float)((2.0 * next_uniform() - 1.0) * bound);
  };
  fill(L.oW1, MLP_H, MLP_IN);
  fill(L.oW2, MLP_H, MLP_H);
  fill(L.oW3, k, MLP_H);
}

// Host weights input-major, outputs padded to whole vectors of 8: W1 [6][64],
// b1, W2 [64][64], b2, W3 [64][kp], b3 [kp] with kp = k rounded up to 8.
static void mlp_pack_host(MlpModel& m) {
  m.packed.clear();
  if (m.k < 1 || m.k > MLP_MAX_K) return;   // a loaded model may be larger: the plain pass takes it
  const MlpLayout L(m.k);
  const int kp = (m.k + 7) / 8 * 8;
  m.packed.assign(MLP_IN * MLP_H + MLP_H + MLP_H * MLP_H + MLP_H + MLP_H * kp + kp, 0.f);
  const float* P = m.params.data();
  float* o = m.packed.data();
  auto layer = [&](int w, int b, int n_in, int n_out, int stride) {
    for (int i = 0; i < n_in; ++i)
      for (int j = 0; j < n_out; ++j) o[i * stride + j] = P[w + j * n_in + i];
    for (int j = 0; j < n_out; ++j) o[n_in * stride + j] = P[b + j];
    o += (n_in + 1) * stride;
  };
  layer(L.oW1, L.ob1, MLP_IN, MLP_H, MLP_H);
  layer(L.oW2, L.ob2, MLP_H, MLP_H, MLP_H);
  layer(L.oW3, L.ob3, MLP_H, m.k, kp);
}

#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
// mlp_forward_argmax with eight outputs of a layer in a vector: each output
// is the same chain of fused multiply-adds over the inputs in the same order,
// hence the same bits and the same pick as the device's.
__attribute__((target("avx2,fma"))) static int mlp_forward_argmax_avx2(const kt_shape& shape,
                                                                       const float* W, int k) {
  alignas(32) float x[MLP_IN], h1[MLP_H], h2[MLP_H], y[MLP_MAX_K];
  shape_features(shape, x);
  const float* w = W;
  const float* in = x;
  const int kp = (k + 7) / 8 * 8;
  const int n_in[3] = {MLP_IN, MLP_H, MLP_H}, n_out[3] = {MLP_H, MLP_H, kp};
  float* outs[3] = {h1, h2, y};
  for (int l = 0; l < 3; ++l) {
    const int n = n_in[l], m = n_out[l];
    for (int j0 = 0; j0 < m; j0 += 32) {   // four chains at a time
      const int nv = (m - j0) / 8 < 4 ? (m - j0) / 8 : 4;
      __m256 acc[4];
      for (int v = 0; v < nv; ++v) acc[v] = _mm256_loadu_ps(w + n * m + j0 + 8 * v);
      for (int i = 0; i < n; ++i) {
        const __m256 a = _mm256_set1_ps(in[i]);
        for (int v = 0; v < nv; ++v)
          acc[v] = _mm256_fmadd_ps(a, _mm256_loadu_ps(w + i * m + j0 + 8 * v), acc[v]);
      }
      for (int v = 0; v < nv; ++v)   // fmaxf(s, 0): max(s, 0) gives 0 for NaN as fmaxf does
        _mm256_storeu_ps(outs[l] + j0 + 8 * v, l < 2 ? _mm256_max_ps(acc[v], _mm256_setzero_ps()) : acc[v]);
    }
    w += (n + 1) * m;
    in = outs[l];
  }
  int best = 0;
  for (int o = 1; o < k; ++o)
    if (y[o] > y[best]) best = o;
  return best;
}

static bool host_has_fma() {
  static const bool v = __builtin_cpu_supports("avx2") && __builtin_cpu_supports("fma");
  return v;
}
#endif

kt_status mlp_upload(Ctx* h, int dtype) {
  SelState& S = h->sel[dtype];
  mlp_pack_host(S.mlp);
  if (h->device < 0) return KT_OK;
  if (S.d_mlp) { (void)hipFree(S.d_mlp); S.d_mlp = nullptr; }
  const size_t pbytes = S.mlp.params.size() * 4, cbytes = S.chosen.size() * 4;
  hipError_t e = hipMalloc(&S.d_mlp, pbytes + cbytes + 256);
  if (e != hipSuccess) { S.d_mlp = nullptr; return hip_fail(h, e, "hipMalloc MLP weights"); }
  e = hipMemcpy(S.d_mlp, S.mlp.params.data(), pbytes, hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy((char*)S.d_mlp + pbytes, S.chosen.data(), cbytes, hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(h, e, "upload MLP weights");
  return KT_OK;
}

kt_status mlp_select_batch(Ctx* h, int dtype, const kt_shape* d_shapes, int32_t n, int32_t* d_ids,
                           hipStream_t st) {
  SelState& S = h->sel[dtype];
  if (!S.d_mlp) return fail(h, KT_ENOTFITTED, "MLP weights not on the device");
  const int k = S.mlp.k;
  const float* P = (const float*)S.d_mlp;
  const int32_t* chosen = (const int32_t*)((const char*)S.d_mlp + S.mlp.params.size() * 4);
  hipLaunchKernelGGL(mlp_select_kernel, dim3((n + 63) / 64), dim3(64), 0, st, d_shapes, n, P, k,
                     chosen, d_ids);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "MLP select launch");
  return KT_OK;
}

// Host selection: the same forward pass on the host copy of the weights, so
// kt_gemm(config_id = -1) with the MLP selector makes no device call besides
// the GEMM launch itself (no copy, no synchronization, capturable in a graph).
kt_status mlp_select_host(Ctx* h, int dtype, const kt_shape* s, int32_t* id) {
  const SelState& S = h->sel[dtype];
  if (S.mlp.params.empty() || S.mlp.k < 1) return fail(h, KT_ENOTFITTED, "no MLP weights");
#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
  // 4992 calls of the C library's fmaf took 6 us of every kt_gemm(-1) call,
  // more than a small kernel; in vectors they take 0.3 us
  if (host_has_fma() && !S.mlp.packed.empty()) {
    *id = S.chosen[mlp_forward_argmax_avx2(*s, S.mlp.packed.data(), S.mlp.k)];
    return KT_OK;
  }
#endif
  *id = S.chosen[mlp_forward_argmax(*s, S.mlp.params.data(), S.mlp.k)];
  return KT_OK;
}

kt_status fit_mlp(Ctx* h, int dtype, const kt_shape* shapes, const int64_t* time_ns, int32_t n,
                  int32_t d, const int32_t* chosen, int32_t k, const kt_mlp_opts* o, void* ws,
                  size_t ws_bytes, hipStream_t st) {
  if (!need_device(h)) return KT_EINVAL;
  if (k > MLP_MAX_K) return fail(h, KT_EINVAL, "MLP supports k <= 64");
  kt_mlp_opts opts = {3000, 1e-3f, nullptr, 13150, 25};
  if (o) opts = *o;
  if (opts.steps < 0 || opts.graph_steps < 0) return fail(h, KT_EINVAL, "negative step count");
  const MlpPlan p = mlp_plan(n, k, d);
  if (!ws || ws_bytes < p.total) return fail(h, KT_EWORKSPACE, "MLP workspace too small");
  char* w = (char*)ws;
  const MlpLayout L(k);
  std::vector<float> P0;
  if (opts.init) P0.assign(opts.init, opts.init + L.total);
  else he_uniform(P0, k, opts.seed);
  hipError_t e = hipMemcpyAsync(w + p.oP, P0.data(), (size_t)L.total * 4, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemsetAsync(w + p.oM, 0, (size_t)L.total * 4, st);
  if (e == hipSuccess) e = hipMemsetAsync(w + p.oV, 0, (size_t)L.total * 4, st);
  if (e == hipSuccess) e = hipMemsetAsync(w + p.oStep, 0, 4, st);
  if (e == hipSuccess) e = hipMemcpyAsync(w + p.oShapes, shapes, (size_t)n * sizeof(kt_shape), hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemcpyAsync(w + p.oT, time_ns, (size_t)n * d * 8, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemcpyAsync(w + p.oChosen, chosen, (size_t)k * 4, hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return hip_fail(h, e, "MLP upload");
  kt_status s = kt_normalize(reinterpret_cast<kt_handle>(h), (const int64_t*)(w + p.oT), n, d,
                             KT_NORM_RELATIVE, (uint16_t*)(w + p.oQ), st);
  if (s != KT_OK) return s;
  hipLaunchKernelGGL(mlp_features_kernel, dim3((n + 255) / 256), dim3(256), 0, st,
                     (const kt_shape*)(w + p.oShapes), n, (float*)(w + p.oX));
  hipLaunchKernelGGL(mlp_targets_kernel, dim3((unsigned)(((int64_t)n * k + 255) / 256)), dim3(256), 0, st,
                     (const uint16_t*)(w + p.oQ), n, d, (const int32_t*)(w + p.oChosen), k,
                     (float*)(w + p.oY));
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(h, e, "MLP data kernels");
  if ((e = set_lds_attr(k)) != hipSuccess) return hip_fail(h, e, "MLP LDS attribute");
  float* P = (float*)(w + p.oP);
  auto one_step = [&](hipStream_t s2) -> hipError_t {
    hipError_t r = launch_fwdbwd(P, (const float*)(w + p.oX), (const float*)(w + p.oY), n, k,
                                 (float*)(w + p.oPart), (float*)(w + p.oPL), nullptr, (int*)(w + p.oStep), s2);
    if (r != hipSuccess) return r;
    hipLaunchKernelGGL(mlp_reduce_adam_kernel, dim3((L.total + 63) / 64), dim3(64), 0, s2, P,
                       (const float*)(w + p.oPart), (const float*)(w + p.oPL), p.nblocks, L.total,
                       nullptr, nullptr, (float*)(w + p.oM), (float*)(w + p.oV),
                       (const int*)(w + p.oStep), opts.lr, 1);
    return hipGetLastError();
  };
  int done = 0;
  if (opts.graph_steps > 1 && opts.steps >= opts.graph_steps) {
    // Capture graph_steps steps once and replay the graph.
    hipStream_t cs = st;
    bool own = false;
    if (cs == nullptr) {
      if ((e = hipStreamCreate(&cs)) != hipSuccess) return hip_fail(h, e, "capture stream");
      own = true;
      if ((e = hipStreamSynchronize(nullptr)) != hipSuccess) return hip_fail(h, e, "sync");
    }
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    for (int i = 0; i < opts.graph_steps && e == hipSuccess; ++i) e = one_step(cs);
    hipError_t e2 = hipStreamEndCapture(cs, &graph);
    if (e == hipSuccess) e = e2;
    if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    while (e == hipSuccess && opts.steps - done >= opts.graph_steps) {
      e = hipGraphLaunch(exec, cs);
      done += opts.graph_steps;
    }
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (own) {
      if (e == hipSuccess) e = hipStreamSynchronize(cs);
      (void)hipStreamDestroy(cs);
    }
    if (e != hipSuccess) return hip_fail(h, e, "MLP training graph");
  }
  for (; done < opts.steps; ++done)
    if ((e = one_step(st)) != hipSuccess) return hip_fail(h, e, "MLP training step");
  std::vector<float> trained(L.total);
  e = hipMemcpyAsync(trained.data(), P, (size_t)L.total * 4, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(h, e, "read MLP weights");
  free_selector_device(h, dtype);
  SelState& S = h->sel[dtype];
  S = SelState();
  S.mlp.k = k;
  S.mlp.params = std::move(trained);
  S.chosen.assign(chosen, chosen + k);
  return mlp_upload(h, dtype);
}

}  // namespace kt

using namespace kt;

extern "C" {

kt_status kt_mlp_workspace_bytes(int32_t n_rows, int32_t n_configs, int32_t k, size_t* bytes) {
  if (!bytes || n_rows < 1 || n_configs < 1 || k < 1 || k > MLP_MAX_K) return KT_EINVAL;
  *bytes = mlp_plan(n_rows, k, n_configs).total;
  return KT_OK;
}

kt_status kt_mlp_num_params(int32_t k, int32_t* n_params) {
  if (!n_params || k < 1 || k > MLP_MAX_K) return KT_EINVAL;
  *n_params = MlpLayout(k).total;
  return KT_OK;
}

kt_status kt_mlp_features(kt_handle hh, const kt_shape* d_shapes, int32_t n, float* d_X, void* stream) {
  Ctx* h = reinterpret_cast<Ctx*>(hh);
  if (!h) return fail(nullptr, KT_EINVAL, "NULL handle");
  if (!need_device(h)) return KT_EINVAL;
  if (n < 0) return fail(h, KT_EINVAL, "n < 0");
  if (n == 0) return KT_OK;
  if (!d_shapes || !d_X) return fail(h, KT_EINVAL, "NULL argument");
  hipLaunchKernelGGL(mlp_features_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                     d_shapes, n, d_X);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "features launch");
  return KT_OK;
}

kt_status kt_mlp_forward_backward(kt_handle hh, const float* d_params, const float* d_X,
                                  const float* d_Y, int32_t n, int32_t k, float* d_pred,
                                  float* d_grad, float* d_loss, void* ws, size_t ws_bytes,
                                  void* stream) {
  Ctx* h = reinterpret_cast<Ctx*>(hh);
  if (!h) return fail(nullptr, KT_EINVAL, "NULL handle");
  if (!need_device(h)) return KT_EINVAL;
  if (n < 1 || k < 1 || k > MLP_MAX_K) return fail(h, KT_EINVAL, "need n >= 1 and 1 <= k <= 64");
  if (!d_params || !d_X) return fail(h, KT_EINVAL, "NULL argument");
  if ((d_grad || d_loss) && !d_Y) return fail(h, KT_EINVAL, "gradients need targets");
  const MlpLayout L(k);
  const int nb = (n + MLP_ROWS - 1) / MLP_ROWS;
  const size_t need = a256((size_t)nb * L.total * 4) + a256((size_t)nb * 4);
  if ((d_grad || d_loss) && (!ws || ws_bytes < need)) return fail(h, KT_EWORKSPACE, "workspace too small");
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = set_lds_attr(k);
  if (e != hipSuccess) return hip_fail(h, e, "MLP LDS attribute");
  float* part = (d_grad || d_loss) ? (float*)ws : nullptr;
  float* pl = part ? (float*)((char*)ws + a256((size_t)nb * L.total * 4)) : nullptr;
  e = launch_fwdbwd(d_params, d_X, (d_grad || d_loss) ? d_Y : nullptr, n, k, part, pl, d_pred, nullptr, st);
  if (e != hipSuccess) return hip_fail(h, e, "forward/backward launch");
  if (part) {
    hipLaunchKernelGGL(mlp_reduce_adam_kernel, dim3((L.total + 63) / 64), dim3(64), 0, st,
                       (float*)nullptr, (const float*)part, (const float*)pl, nb, L.total, d_grad,
                       d_loss, (float*)nullptr, (float*)nullptr, (const int*)nullptr, 0.f, 0);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(h, e, "gradient reduction launch");
  }
  return KT_OK;
}

kt_status kt_get_mlp(kt_handle hh, kt_dtype dtype, int32_t* n_params, float* params) {
  Ctx* h = reinterpret_cast<Ctx*>(hh);
  if (!h) return fail(nullptr, KT_EINVAL, "NULL handle");
  if ((int)dtype < 0 || (int)dtype >= NUM_DTYPES) return fail(h, KT_EINVAL, "bad dtype");
  if (!n_params) return fail(h, KT_EINVAL, "NULL n_params");
  const SelState& S = h->sel[dtype];
  if (S.kind != KT_SEL_MLP) return fail(h, KT_ENOTFITTED, "no MLP fitted");
  *n_params = (int32_t)S.mlp.params.size();
  if (params) memcpy(params, S.mlp.params.data(), S.mlp.params.size() * 4);
  return KT_OK;
}

}  // extern "C"
