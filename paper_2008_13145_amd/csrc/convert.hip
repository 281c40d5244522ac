// Operand conversions for the low-precision GEMM paths.
//
// BF16: round to nearest even of the FP32 bit pattern, NaN kept quiet.
// FP8 e4m3 (OCP "e4m3fn", largest finite 448): per-tensor scale
// s = 448 / amax(|x|) in FP32 (s = 1 when amax = 0), code = e4m3(x * s) with
// the product rounded to FP32, round to nearest even, saturating to +-448,
// NaN -> 0x7F.  amax is an order-independent atomic maximum of the
// non-negative float bit patterns, so the scale is exact and deterministic.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kt_internal.hpp"

namespace kt {

// All three passes are HBM-bound and take 16 elements a thread and step, in
// 16-byte loads and stores, when both buffers lie on 16-byte boundaries (the
// elements after the last 16, and other buffers, one by one).
// 4096 x 4096: BF16 17.2 -> 15.3 us, FP8 (both passes) 70.6 -> 32.6 us.
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t bf16_of(float x) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (u >> 16) | 0x40u;
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__global__ void __launch_bounds__(256)
cvt_bf16_kernel(const float* __restrict__ x, uint16_t* __restrict__ y, int64_t n, int64_t nv) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = tid; v < nv; v += stride) {   // 8 elements: two loads, one store
    const f32x4v a = reinterpret_cast<const f32x4v*>(x)[2 * v], b = reinterpret_cast<const f32x4v*>(x)[2 * v + 1];
    u32x4v o;
    o[0] = bf16_of(a[0]) | (bf16_of(a[1]) << 16);
    o[1] = bf16_of(a[2]) | (bf16_of(a[3]) << 16);
    o[2] = bf16_of(b[0]) | (bf16_of(b[1]) << 16);
    o[3] = bf16_of(b[2]) | (bf16_of(b[3]) << 16);
    reinterpret_cast<u32x4v*>(y)[v] = o;
  }
  for (int64_t i = 8 * nv + tid; i < n; i += stride) y[i] = (uint16_t)bf16_of(x[i]);
}

__global__ void zero_u32_kernel(uint32_t* p) { *p = 0u; }

// |x| as bits: NaN sorts above infinity.
__device__ __forceinline__ uint32_t abs_bits(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }

__global__ void __launch_bounds__(256)
amax_kernel(const float* __restrict__ x, int64_t n, int64_t nv, uint32_t* __restrict__ amax_bits) {
  __shared__ uint32_t red[4];
  uint32_t m = 0u;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
#pragma unroll 4
  for (int64_t v = tid; v < nv; v += stride) {
    const f32x4v a = reinterpret_cast<const f32x4v*>(x)[v];
    m = max(m, max(max(abs_bits(a[0]), abs_bits(a[1])), max(abs_bits(a[2]), abs_bits(a[3]))));
  }
  for (int64_t i = 4 * nv + tid; i < n; i += stride) m = max(m, abs_bits(x[i]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = max(max(red[0], red[1]), max(red[2], red[3]));
    // the word only grows: work-groups that cannot raise it leave it alone
    if (m > __hip_atomic_load(amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(amax_bits, m);
  }
}

__device__ __forceinline__ float fp8_scale_of(uint32_t amax_bits) {
  const float amax = __uint_as_float(amax_bits);
  return amax > 0.f ? 448.0f / amax : 1.0f;
}

// Two codes in the low 16 bits: saturate, then round to nearest even.
__device__ __forceinline__ uint32_t fp8_pair(float a, float b) {
  const float ca = fminf(fmaxf(a, -448.0f), 448.0f), cb = fminf(fmaxf(b, -448.0f), 448.0f);
  uint32_t c = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(ca, cb, 0, false) & 0xFFFFu;
  if (a != a) c = (c & 0xFF00u) | 0x7Fu;
  if (b != b) c = (c & 0x00FFu) | 0x7F00u;
  return c;
}

__global__ void __launch_bounds__(256)
quant_fp8_kernel(const float* __restrict__ x, int64_t n, int64_t nv,
                 const uint32_t* __restrict__ amax_bits, uint8_t* __restrict__ y,
                 float* __restrict__ scale_out) {
  const float s = fp8_scale_of(*amax_bits);
  if (blockIdx.x == 0 && threadIdx.x == 0) *scale_out = s;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = tid; v < nv; v += stride) {   // 16 elements: four loads, one store
    u32x4v o;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4v a = reinterpret_cast<const f32x4v*>(x)[4 * v + q];
      o[q] = fp8_pair(a[0] * s, a[1] * s) | (fp8_pair(a[2] * s, a[3] * s) << 16);
    }
    reinterpret_cast<u32x4v*>(y)[v] = o;
  }
  for (int64_t i = 16 * nv + tid; i < n; i += stride) y[i] = (uint8_t)fp8_pair(x[i] * s, 0.0f);
}

// Up to SMALL_N elements in one work-group, which holds them in registers between
// the two passes: one launch instead of three.  4096 elements take 3.9 us on the
// stream instead of 8.9, 48000 5.9 instead of 9.9, 65536 7.1 instead of 9.7; one CU's
// loads cost 1 us per 10000 elements, so at 100000 the three kernels are ahead.
constexpr int SMALL_THREADS = 1024, SMALL_CHUNKS = 16, SMALL_N = SMALL_THREADS * SMALL_CHUNKS * 4;

__global__ void __launch_bounds__(SMALL_THREADS)
quant_fp8_small_kernel(const float* __restrict__ x, int n, uint32_t* __restrict__ amax_bits,
                       uint8_t* __restrict__ y, float* __restrict__ scale_out) {
  __shared__ uint32_t red[SMALL_THREADS / 64];
  const int tid = threadIdx.x, nv = n / 4, rest = 4 * nv + tid;
  f32x4v a[SMALL_CHUNKS];
  uint32_t m = 0u;
#pragma unroll
  for (int i = 0; i < SMALL_CHUNKS; ++i) {
    const int v = tid + i * SMALL_THREADS;
    a[i] = v < nv ? reinterpret_cast<const f32x4v*>(x)[v] : f32x4v{0.f, 0.f, 0.f, 0.f};
  }
  const float last = rest < n ? x[rest] : 0.f;
#pragma unroll
  for (int i = 0; i < SMALL_CHUNKS; ++i)
    m = max(m, max(max(abs_bits(a[i][0]), abs_bits(a[i][1])), max(abs_bits(a[i][2]), abs_bits(a[i][3]))));
  m = max(m, abs_bits(last));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o));
  if ((tid & 63) == 0) red[tid >> 6] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < SMALL_THREADS / 64; ++w) m = max(m, red[w]);
  const float s = fp8_scale_of(m);
  if (tid == 0) {
    *amax_bits = m;
    *scale_out = s;
  }
#pragma unroll
  for (int i = 0; i < SMALL_CHUNKS; ++i) {
    const int v = tid + i * SMALL_THREADS;
    if (v < nv)
      reinterpret_cast<uint32_t*>(y)[v] = fp8_pair(a[i][0] * s, a[i][1] * s) | (fp8_pair(a[i][2] * s, a[i][3] * s) << 16);
  }
  if (rest < n) y[rest] = (uint8_t)fp8_pair(last * s, 0.0f);
}

// Work-groups for n threads' worth of steps, at most `most`.
static unsigned grid_for(int64_t n, int64_t most) {
  const int64_t b = (n + 255) / 256;
  return (unsigned)(b < most ? (b > 0 ? b : 1) : most);
}

static bool on16(const void* p, const void* q) { return (((uintptr_t)p | (uintptr_t)q) & 15u) == 0; }

}  // namespace kt

using namespace kt;

extern "C" {

kt_status kt_convert_bf16(kt_handle hh, const float* x, int64_t n, uint16_t* y, void* stream) {
  Ctx* h = reinterpret_cast<Ctx*>(hh);
  if (!h) return fail(nullptr, KT_EINVAL, "NULL handle");
  if (!need_device(h)) return KT_EINVAL;
  if (n < 0) return fail(h, KT_EINVAL, "n < 0");
  if (n == 0) return KT_OK;
  if (!x || !y) return fail(h, KT_EINVAL, "NULL buffer");
  const int64_t nv = on16(x, y) ? n / 8 : 0;
  hipLaunchKernelGGL(cvt_bf16_kernel, dim3(grid_for(nv > 0 ? nv : n, 4096)), dim3(256), 0,
                     (hipStream_t)stream, x, y, n, nv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "BF16 conversion launch");
  return KT_OK;
}

kt_status kt_quantize_fp8(kt_handle hh, const float* x, int64_t n, uint8_t* y, float* d_scale,
                          void* workspace, size_t ws_bytes, void* stream) {
  Ctx* h = reinterpret_cast<Ctx*>(hh);
  if (!h) return fail(nullptr, KT_EINVAL, "NULL handle");
  if (!need_device(h)) return KT_EINVAL;
  if (n < 0) return fail(h, KT_EINVAL, "n < 0");
  if (!d_scale) return fail(h, KT_EINVAL, "NULL scale");
  if (n > 0 && (!x || !y)) return fail(h, KT_EINVAL, "NULL buffer");
  if (!workspace || ws_bytes < 4) return fail(h, KT_EWORKSPACE, "FP8 quantization needs 4 bytes of workspace");
  hipStream_t st = (hipStream_t)stream;
  uint32_t* amax = (uint32_t*)workspace;
  if (n > 0 && n <= SMALL_N && on16(x, y)) {
    hipLaunchKernelGGL(quant_fp8_small_kernel, dim3(1), dim3(SMALL_THREADS), 0, st, x, (int)n, amax, y, d_scale);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(h, e, "FP8 quantization launch");
    return KT_OK;
  }
  hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(1), 0, st, amax);
  // one atomic per work-group: four a CU are enough to keep the loads in flight
  const int64_t na = on16(x, nullptr) ? n / 4 : 0;
  if (n > 0)
    hipLaunchKernelGGL(amax_kernel, dim3(grid_for(na > 0 ? na : n, 1024)), dim3(256), 0, st, x, n, na,
                       amax);
  const int64_t nv = on16(x, y) ? n / 16 : 0;
  hipLaunchKernelGGL(quant_fp8_kernel, dim3(grid_for(nv > 0 ? nv : n, 4096)), dim3(256), 0, st, x, n,
                     nv, (const uint32_t*)amax, y, d_scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "FP8 quantization launch");
  return KT_OK;
}

}  // extern "C"
