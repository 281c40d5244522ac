// Low-precision GEMM family for gfx950: BF16 or FP8-e4m3 inputs, FP32
// accumulation and output.  C_b = alpha * s * op(A_b) * op(B_b) + beta * C_b
// with s = 1 for BF16 and s = 1 / (scaleA * scaleB) for per-tensor-scaled FP8.
//
// Same configuration knobs as the FP32 family (work-group tile BM x BN, per
// wave an (8T) x (8T) block, K depth BK per LDS stage), with T in
// {2, 4, 8, 16}: T = 2 is one 16x16 MFMA block per wave (16x16x32 BF16,
// 16x16x128 FP8), T = 4 one 32x32 block, T = 8 a 2x2 and T = 16 a 4x4 grid
// of them (the 4x4 grid keeps its 256 accumulators in AGPRs and halves the
// LDS bytes read per MFMA against the 2x2 grid).
// BF16 runs v_mfma_f32_32x32x16_bf16 (8 consecutive K values per lane, lane
// l: row l % 32, K offset 8 * (l / 32)); FP8 runs the 64-deep
// v_mfma_scale_f32_32x32x64_f8f6f4 with unit block scales (32 K bytes per
// lane, K offset 32 * (l / 32)).  A and B fragments take K in the same lane
// order, so each product pairs the right elements whatever order the unit
// sums them in.  How tiles reach LDS and fragments are read: gemm_lp_dma.hpp.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gemm_f32.hpp"

namespace kt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

template <int EB>   // element bytes: 2 = BF16, 1 = FP8 e4m3
struct LpElem;
template <>
struct LpElem<2> { typedef uint16_t T; static constexpr int KSTEP = 16, KSTEP16 = 32; };
template <>
struct LpElem<1> { typedef uint8_t T; static constexpr int KSTEP = 64, KSTEP16 = 128; };

template <int EB, int BM, int BN, int T, int BK, int TA, int TB>
struct GemmLpCfg {
  static constexpr int WT = 8 * T;
  // T = 2 runs the 16x16 MFMAs (16x16x32 BF16, 16x16x128 FP8), larger T the
  // 32x32 ones (32x32x16 BF16, 32x32x64 FP8).
  static constexpr int MB = T == 2 ? 16 : 32;        // MFMA block edge
  static constexpr int SUB = WT / MB;                // MFMA blocks per wave edge
  static constexpr int KSTEP = T == 2 ? LpElem<EB>::KSTEP16 : LpElem<EB>::KSTEP;
  static constexpr int WAVES_N = BN / WT;
  static constexpr int WAVES = (BM / WT) * WAVES_N;
  static constexpr int NT = WAVES * 64;
  static_assert(T == 2 || T == 4 || T == 8 || T == 16, "low-precision wave blocks of 16 to 128");
  static_assert(BM % WT == 0 && BN % WT == 0, "tile must hold whole wave blocks");
  static_assert(WAVES >= 1 && WAVES <= 16, "1..16 waves per work-group");
  static_assert(BK % KSTEP == 0, "BK multiple of the MFMA depth");
};

// One lane's operand fragment for one MFMA: 8 BF16 values (16 bytes) or
// 32 FP8 codes (32 bytes).
template <int EB>
struct LpFrag;
template <>
struct LpFrag<2> { bf16x8 v; };
template <>
struct LpFrag<1> { i32x8 v; };

__device__ __forceinline__ void lp_mfma(const LpFrag<2>& a, const LpFrag<2>& b, f32x16& c) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, c, 0, 0, 0);
}

// Operand formats 0 / 0 = e4m3 for A and B; block scales 127 = 2^0 (E8M0).
__device__ __forceinline__ void lp_mfma(const LpFrag<1>& a, const LpFrag<1>& b, f32x16& c) {
  c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a.v, b.v, c, 0, 0, 0, 127, 0, 127);
}

__device__ __forceinline__ void lp_mfma(const LpFrag<2>& a, const LpFrag<2>& b, f32x4& c) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}

__device__ __forceinline__ void lp_mfma(const LpFrag<1>& a, const LpFrag<1>& b, f32x4& c) {
  c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a.v, b.v, c, 0, 0, 0, 127, 0, 127);
}

}  // namespace kt
