// LDS-DMA pipeline of the FP32 family (T = 2, 4, 8), taken when every
// operand row starts on a 4-byte boundary and holds a 16-byte chunk
// (launch_gemm_f32); no 16-byte read leaves an operand.
// Same configuration knobs and results contract as gemm_f32.hpp; the
// differences:
//
// * Tiles move HBM -> LDS by global_load_lds_dwordx4 (1 KiB per wave
//   instruction), NS = 2..4 stages in flight, waited for with vmcnt; no
//   register staging and no LDS stores by the waves.
// * Each operand keeps its stored layout in LDS: K-contiguous operands as
//   [row][k] with 16-byte chunks XOR-swizzled by row (as the low-precision
//   tiles), M/N-contiguous ones as [k][col].
// * T = 8 with BK >= 16 multiplies on the BF16 matrix cores (SplitFrag below).
// * The MFMA's K positions are assigned by lane group instead of
//   interleaved: for the 32x32x2 MFMA lane half h takes k = h * BK / 2 + q at
//   step q, for the 16x16x4 MFMA lane quarter g takes k = g * BK / 4 + q, so a
//   lane reads consecutive k of one row of a K-contiguous tile.  A and B use
//   the same assignment, so each product pairs matching elements; the sums
//   run in another order than the register-staged kernel's (same bound).
#pragma once
#include "gemm_lp_dma.hpp"

namespace kt {

template <int BM, int BN, int T, int BK, int TA, int TB>
struct F32DmaCfg {
  using Base = GemmF32Cfg<BM, BN, T, BK, TA, TB>;
  static constexpr int NT = Base::NT, WAVES = Base::WAVES, WT = Base::WT;
  static constexpr int A_BYTES = BM * BK * 4, B_BYTES = BN * BK * 4;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int BUDGET = 64 * 1024;
  static constexpr int NS_FIT = BUDGET / STAGE;
  static constexpr int NS = NS_FIT < 2 ? 2 : (NS_FIT > 4 ? 4 : NS_FIT);
  static constexpr int LDS_BYTES = NS * STAGE;
  static constexpr int NBA = A_BYTES / 1024, NBB = B_BYTES / 1024;
  static constexpr int NBLK = NBA + NBB;
  static constexpr int NW_LO = NBLK / WAVES, NW_HI = (NBLK + WAVES - 1) / WAVES;
  // a K-major row is BK floats: 2..16 chunks of 16 bytes
  static constexpr int KCPR = BK / 4;
  static_assert(T >= 2, "the 4x4x1 family keeps the register-staged pipeline");
  static_assert(A_BYTES % 1024 == 0 && B_BYTES % 1024 == 0, "tiles of whole 1 KiB blocks");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
  static_assert((NS - 2) * NW_HI < 64, "vmcnt range");
  // An M/N-contiguous row must be whole chunks; a 1 KiB block must hold whole rows.
  static_assert((BM * 4) % 16 == 0 && (BN * 4) % 16 == 0, "whole chunks per row");
};

// M/N-major FP32 rows (one k each, COLS floats = CPR 16-byte chunks): the
// lane groups of an MFMA step read the same columns of rows BK/2 apart
// (32x32x2: two halves of 32 lanes, 128 bytes each) or BK/4 apart (16x16x4:
// four quarters of 16 lanes, 64 bytes each), which would fall on the same
// banks of a 256-byte bank line; XOR-ing a group's chunk index by 8 (halves)
// or by 4 x its quarter (quarters) puts the groups on different banks.
template <int CPR, int BK, int T>
__device__ __forceinline__ int f32_mswz(int k) {
  if constexpr (T == 2) return CPR >= 8 ? (((k / (BK / 4)) & 3) * 4) % CPR : 0;
  else return CPR >= 16 ? ((k / (BK / 2)) & 1) * 8 : 0;
}

template <int BM, int BN, int T, int BK>
struct F32Swz {
  __device__ __forceinline__ static int k(int r) { return kswz<BK / 4>(r); }
  __device__ __forceinline__ static int mn_a(int r) { return f32_mswz<BM / 4, BK, T>(r); }
  __device__ __forceinline__ static int mn_b(int r) { return f32_mswz<BN / 4, BK, T>(r); }
};

template <int BM, int BN, int T, int BK, int TA, int TB>
__device__ __forceinline__ void f32_dma_zero_tail(char* stage, int kvalid, int tid) {
  using Cfg = F32DmaCfg<BM, BN, T, BK, TA, TB>;
  asm volatile("" : "+s"(kvalid));   // keeps this rarely run arithmetic out of the stage loop's preheader
  tid = rarely(tid);
#pragma unroll
  for (int op = 0; op < 2; ++op) {
    const bool kmajor = op == 0 ? (TA == 0) : (TB == 1);
    const int cols = op == 0 ? BM : BN;
    float* t = reinterpret_cast<float*>(stage + (op == 0 ? 0 : Cfg::A_BYTES));
    if (kmajor) {
      constexpr int CPR = Cfg::KCPR;
      for (int i = tid; i < cols * CPR; i += Cfg::NT) {
        const int r = i / CPR, c = i % CPR;
        f32x4* p = reinterpret_cast<f32x4*>(t + r * BK) + (c ^ kswz<CPR>(r));
        const int from = kvalid - 4 * c;   // first element to clear
        if (from <= 0) *p = f32x4{0.f, 0.f, 0.f, 0.f};
        else
          for (int e = from; e < 4; ++e) (*p)[e] = 0.f;
      }
    } else {
      for (int i = kvalid * cols / 4 + tid; i < BK * cols / 4; i += Cfg::NT)
        reinterpret_cast<f32x4*>(t)[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
}

// Element (row, k) of a K-major tile / (k, col) of an M/N-major tile.
template <int BK>
__device__ __forceinline__ float f32_at_kmajor(const float* t, int row, int k) {
  return t[row * BK + ((k >> 2) ^ kswz<BK / 4>(row)) * 4 + (k & 3)];
}
template <int COLS, int BK, int T>
__device__ __forceinline__ float f32_at_mnmajor(const float* t, int k, int col) {
  constexpr int CPR = COLS / 4;
  return t[k * COLS + (((col >> 2) ^ f32_mswz<CPR, BK, T>(k)) << 2) + (col & 3)];
}

// FP32 products on the BF16 matrix cores (T = 8 with BK >= 16).  A float
// of 2^-110 or more is exactly the sum of three BF16 values, x = h + m + l (each
// the rounding of what is left: 24 bits as 8 + 8 + 8; below, the last piece ends
// at BF16's smallest subnormal and 2^-134 may be left), and
//   a b = ah bh + (ah bm + am bh) + (ah bl + am bm + al bh) + terms < 2^-24 |a b| in all,
// so six BF16 MFMAs, whose products are exact and whose sums are FP32, take
// the place of the eight times slower FP32 ones.  Each 16-deep step adds the
// small products first.  The result is nearer to the exact product than the
// FP32 MFMA's, which rounds after every k: relative error against FP64 of
// normal operands at K = 16 / 128 / 1024 / 4096: 3.4e-8 / 1.65e-7 / 4.9e-7 /
// 1.00e-6, with FP32 MFMAs 7.3e-8 / 2.04e-7 / 5.7e-7 / 1.15e-6.  (Truncated
// instead of rounded pieces bias the sums: 9.5e-6 for positive operands at
// K = 4096.)  Below K = 5 the six sums round more often than the few FP32
// ones: products with K < 16 keep the FP32 MFMAs (launch_gemm_f32).
//
// A lane splits (64 + 64) * 16 / 64 values for 24 MFMAs a step: about 200
// vector instructions (800 clocks) beside 768 clocks of MFMA, so the split of
// step g + 1 is placed between the MFMAs of step g; one after the other the
// two took turns.  Counters at 4096^3: MFMA busy 51 to 53 % of cycles at 1.8 to 1.95
// GHz, to which the clock falls under this load.  Subtraction with a shift, not
// v_dot2_f32_bf16, makes the residuals: the dot unit shares the matrix pipe.
// 32x32 wave blocks (T = 4) split twice as many values per MFMA and gained
// nothing.  128x128 tiles, BK = 32, with FP32 MFMAs -> this way on one card:
// 4096^3 NT 1090 -> 776 us (126 -> 177 TFLOP/s), NN 1127 -> 777 us; 2048x1024x1536
// batch 16 TN 880 -> 620 us.
//
// Two kinds of operand do not split: infinities and values that round to
// infinity in BF16, whose residual is NaN, and values below 2^-110 (a NaN does:
// its row or column of the product is NaN either way).  A work-group that
// meets either where it shows (a non-finite sum that no NaN explains; a sum
// below 2^27 times what its operands' pieces may leave out of it, where any
// left something out: one OR per two values, 2.5 % of the kernel) computes its
// tile again on FP32 MFMAs, through the same stages.  In products of 32 stages
// or more it leaves the split out when the first stage holds an infinity or a
// value of 2^62 or more (smaller ones seldom overflow; looking costs 3 % of 16
// stages).  4096^3 NT / TN with infinities on 128x128 tiles: 0.96 / 1.08 ms where
// the first stage shows them, 1.75 / 1.79 ms where a later one does (FP32 kernels
// 1.04; the second pass straight from memory, 8 of K at a time: 1.20 / 1.46 and
// 1.72 / 1.94); 64x64 tiles 1.73 / 1.82 and 2.84 / 3.02 (from memory, 2 at a time: 5.5).
// With NaN 0.74 / 0.73.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// The larger value, NaN if either is (a single three-operand instruction
// where two are nested).
__device__ __forceinline__ float largest(float a, float b) { return __builtin_elementwise_maximum(a, b); }

struct SplitFrag {
  bf16x8 h, m, l;

  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(h), "+v"(m), "+v"(l)); }
  __device__ __forceinline__ static float low(bf16x2 v) {
    return __uint_as_float(__builtin_bit_cast(uint32_t, v) << 16);
  }
  __device__ __forceinline__ static float high(bf16x2 v) {
    return __uint_as_float(__builtin_bit_cast(uint32_t, v) & 0xffff0000u);
  }

  // Values 2 p and 2 p + 1; most collects the largest magnitude, NaN above all,
  // left the bits of what the first two pieces leave: the third takes it
  // whole unless one of the lower 16 is set.
  __device__ __forceinline__ void set(int p, const float a, const float b, float& most, uint32_t& left) {
    most = largest(most, largest(__builtin_fabsf(a), __builtin_fabsf(b)));
    const bf16x2 hp = __builtin_convertvector(f32x2{a, b}, bf16x2);
    const float ra = a - low(hp), rb = b - high(hp);   // exact
    const bf16x2 mp = __builtin_convertvector(f32x2{ra, rb}, bf16x2);
    const float qa = ra - low(mp), qb = rb - high(mp);
    // (asm: reassociated by the compiler, the chain of ORs keeps its inputs in registers)
    asm("v_or3_b32 %0, %0, %1, %2" : "+v"(left) : "v"(qa), "v"(qb));
    const bf16x2 lp = __builtin_convertvector(f32x2{qa, qb}, bf16x2);
    h[2 * p] = hp[0]; h[2 * p + 1] = hp[1];
    m[2 * p] = mp[0]; m[2 * p + 1] = mp[1];
    l[2 * p] = lp[0]; l[2 * p + 1] = lp[1];
  }
};

template <int T, int BK>
struct F32Split {
  static constexpr bool value = T == 8 && BK >= 16;
};

// Stages from which on a split kernel looks through its first one (SplitFrag).
constexpr int F32_LOOK_FIRST = 32;

// At least two waves per SIMD for the split kernels: with that register
// budget the accumulators stay out of the AGPRs (and of copies to and from
// them).  Not where it spills in the stage loop: tiles of two waves, 32 deep,
// both operands M/N-major, have twelve block offsets and 32 single LDS reads a
// step.
template <int BM, int BN, int T, int BK, int TA, int TB>
struct F32DmaOcc {
  static constexpr bool SPILLS = BM * BN == 2 * 64 * 64 && BK == 32 && TA == 1 && TB == 0;
  static constexpr int value = F32Split<T, BK>::value && !SPILLS ? 2 : 1;
};

template <int BM, int BN, int T, int BK, int TA, int TB>
__global__ void __launch_bounds__(BM * BN / (T * T))
__attribute__((amdgpu_waves_per_eu(F32DmaOcc<BM, BN, T, BK, TA, TB>::value, 8)))
gemm_f32_dma_kernel(GemmArgs args) {
  using Cfg = F32DmaCfg<BM, BN, T, BK, TA, TB>;
  constexpr int NS = Cfg::NS;
  constexpr int WT = Cfg::WT;
  __shared__ __attribute__((aligned(16))) char lds[Cfg::LDS_BYTES];
  __shared__ int leave[2];   // split kernels: the first stage, or a sum, asks for FP32 MFMAs

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = Cfg::WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lds0 = lds_address(lds);
  const int wm0 = (wave / Cfg::Base::WAVES_N) * WT;
  const int wn0 = (wave % Cfg::Base::WAVES_N) * WT;
  int tm, tn;
  int64_t bz;
  load_args(args);
  block_coords(blockIdx.x, args, tm, tn, bz);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int64_t M = args.M, N = args.N, K = args.K;
  DmaSource<Cfg, 4, BM, BN, BK, TA, TB, F32Swz<BM, BN, T, BK>> src;

  auto A_at = [&](const float* t, int m, int k) {
    if constexpr (TA == 0) return f32_at_kmajor<BK>(t, m, k);
    else return f32_at_mnmajor<BM, BK, T>(t, k, m);
  };
  auto B_at = [&](const float* t, int n, int k) {
    if constexpr (TB == 1) return f32_at_kmajor<BK>(t, n, k);
    else return f32_at_mnmajor<BN, BK, T>(t, k, n);
  };
  // Four consecutive k (k0 a multiple of 4) of one row / column: one 16-byte
  // LDS read from a K-major tile (a whole swizzled chunk), four from an
  // M/N-major one.
  auto A4 = [&](const float* t, int m, int k0) {
    if constexpr (TA == 0)
      return *reinterpret_cast<const f32x4*>(t + m * BK + ((k0 >> 2) ^ kswz<BK / 4>(m)) * 4);
    else
      return f32x4{A_at(t, m, k0), A_at(t, m, k0 + 1), A_at(t, m, k0 + 2), A_at(t, m, k0 + 3)};
  };
  auto B4 = [&](const float* t, int n, int k0) {
    if constexpr (TB == 1)
      return *reinterpret_cast<const f32x4*>(t + n * BK + ((k0 >> 2) ^ kswz<BK / 4>(n)) * 4);
    else
      return f32x4{B_at(t, n, k0), B_at(t, n, k0 + 1), B_at(t, n, k0 + 2), B_at(t, n, k0 + 3)};
  };

  constexpr int NACC = (T == 2) ? 4 : (T == 4) ? 16 : 1;
  constexpr bool SPLIT = F32Split<T, BK>::value;
  constexpr int SUB = 2;   // T = 8: 32x32 blocks per wave edge
  float acc[NACC];
  float total[T == 2 ? 4 : 1] = {};
#pragma unroll
  for (int i = 0; i < NACC; ++i) acc[i] = 0.f;
  f32x16 sacc[SUB][SUB];   // T = 8
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < SUB; ++i)
#pragma unroll
      for (int j = 0; j < SUB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[i][j][r] = 0.f;
  };
  if constexpr (T == 8) clear();

  const int nk = (int)((K + BK - 1) / BK);
  const int my_blocks = (wave < Cfg::NBLK % Cfg::WAVES || Cfg::NBLK % Cfg::WAVES == 0)
                            ? Cfg::NW_HI : Cfg::NW_LO;
  auto start = [&](int wave, int lane) __attribute__((always_inline)) {
    src.init(args, static_cast<const char*>(args.A) + bz * args.sA * 4,
             static_cast<const char*>(args.B) + bz * args.sB * 4, m0, n0, wave, lane);
#pragma nounroll
    for (int s = 0; s < NS - 1; ++s)
      if (s < nk) src.issue(args, m0, n0, lds0 + s * Cfg::STAGE);
  };

  // Make stage kt readable: its DMA has landed for every wave, K beyond the
  // product is zero, and the stage AHEAD stages on is on its way into the
  // buffer that every wave has finished reading.
  auto open_stage = [&](int kt, int issued, int ahead_max) __attribute__((always_inline)) {
    const int ahead = min(ahead_max, nk - 1 - kt);
    if (my_blocks == Cfg::NW_HI) wait_stage<Cfg::NW_HI, NS>(ahead);
    else wait_stage<Cfg::NW_LO, NS>(ahead);
    char* cur = lds + (kt % NS) * Cfg::STAGE;
    if (kt == nk - 1 && src.settle(args, m0, n0, (int)(K - (int64_t)kt * BK), cur, tid))
      vm_wait_barrier<0>();
    if (kt == nk - 1 && K - (int64_t)kt * BK < BK) {
      f32_dma_zero_tail<BM, BN, T, BK, TA, TB>(cur, (int)(K - (int64_t)kt * BK), tid);
      vm_wait_barrier<0>();
    }
    if (issued < nk) src.issue(args, m0, n0, lds0 + (issued % NS) * Cfg::STAGE);
  };
  // The product on the BF16 matrix cores; false where it has to be done with
  // FP32 MFMAs instead (for the whole work-group alike, which is then done
  // with its LDS).
  auto split_product = [&]() __attribute__((always_inline)) {
    // 32x32x16 MFMAs: lane half h takes k = h * BK / 2 + 8 s .. + 7 at step s.
    // The fragments of step g + 1 are read and split while the MFMAs of step
    // g run.
    constexpr int S = BK / 16;   // steps per stage
    const int r32 = lane & 31, h = lane >> 5;
    const int steps = nk * S;
    float most_a[SUB] = {0.f, 0.f}, most_b[SUB] = {0.f, 0.f};   // largest magnitude of each row and column
    uint32_t left = 0u;   // a lower half that is not zero: a value that does not split
    struct Frags { SplitFrag a[SUB], b[SUB]; };
    Frags f0, f1;
    f32x4 xa[SUB][2], xb[SUB][2];
    auto fetch = [&](int g) {
      const char* cur = lds + ((g / S) % NS) * Cfg::STAGE;
      const float* as = reinterpret_cast<const float*>(cur);
      const float* bs = reinterpret_cast<const float*>(cur + Cfg::A_BYTES);
      const int k = h * (BK / 2) + 8 * (g % S);
#pragma unroll
      for (int i = 0; i < SUB; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          xa[i][q] = A4(as, wm0 + 32 * i + r32, k + 4 * q);
          xb[i][q] = B4(bs, wn0 + 32 * i + r32, k + 4 * q);
        }
    };
    // pair u (0 .. 8 SUB - 1) of the fetched values: 4 of each fragment
    auto split = [&](Frags& f, int u) {
      const int i = u / 8, p = u % 4;
      if (u % 8 < 4) f.a[i].set(p, xa[i][p / 2][2 * (p % 2)], xa[i][p / 2][2 * (p % 2) + 1], most_a[i], left);
      else f.b[i].set(p, xb[i][p / 2][2 * (p % 2)], xb[i][p / 2][2 * (p % 2) + 1], most_b[i], left);
    };
    // MFMA u of a step: six products, the small ones first, of every block
    auto mfma = [&](const Frags& f, int u) {
      const int i = u / SUB % SUB, j = u % SUB, w = u / (SUB * SUB);
      const bf16x8 a = w == 0 ? f.a[i].l : (w == 2 || w == 3) ? f.a[i].m : f.a[i].h;
      const bf16x8 b = w == 1 ? f.b[j].l : (w == 2 || w == 4) ? f.b[j].m : f.b[j].h;
      sacc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, sacc[i][j], 0, 0, 0);
    };
    constexpr int NM = 6 * SUB * SUB, NP = 8 * SUB;
    constexpr int LEAD = NM - NP > 0 ? NM - NP : 0;   // MFMAs over the latency of the reads
    auto step = [&](const Frags& cur, Frags& next, int g) __attribute__((always_inline)) {
      if (g % S == 0) open_stage(g / S, g / S + NS - 1, NS - 2);
      fetch(g);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < LEAD; ++u) mfma(cur, u);
#pragma unroll
      for (int u = 0; u < (NM - LEAD > NP ? NM - LEAD : NP); ++u) {
        __builtin_amdgcn_sched_barrier(0);
        if (LEAD + u < NM) mfma(cur, LEAD + u);
        if (u < NP) split(next, u);
      }
#pragma unroll
      for (int i = 0; i < SUB; ++i) {   // done here, not sunk to their use in the next step
        next.a[i].pin();
        next.b[i].pin();
      }
    };
    auto last = [&](const Frags& cur) {
#pragma unroll
      for (int u = 0; u < NM; ++u) mfma(cur, u);
    };
    // true in every wave when one of them says so
    auto any_wave = [&](bool v, int flag) __attribute__((always_inline)) {
      if constexpr (Cfg::WAVES == 1) {
        return (bool)__any(v);
      } else {
        if (__any(v) && lane == 0) leave[flag] = 1;
        vm_wait_barrier<63>();   // the flag; transfers stay in flight
        return __builtin_amdgcn_readfirstlane(leave[flag]) != 0;
      }
    };
    if (Cfg::WAVES > 1 && tid == 0) leave[0] = leave[1] = 0;
    open_stage(0, NS - 1, NS - 2);
    fetch(0);
    if (nk >= F32_LOOK_FIRST) {
      // only rows and columns of the product count (below, too): beyond them
      // lies whatever the operands' memory holds
      bool large = false;
#pragma nounroll
      for (int g = S - 1; g >= 0; --g) {
        fetch(g);
#pragma unroll
        for (int i = 0; i < SUB; ++i) {
          float ma = 0.f, mb = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            ma = largest(ma, __builtin_fabsf(xa[i][e / 4][e % 4]));
            mb = largest(mb, __builtin_fabsf(xb[i][e / 4][e % 4]));
          }
          large = large || (32 * i + r32 < M - m0 - wm0 && ma >= 0x1p62f) ||
                  (32 * i + r32 < N - n0 - wn0 && mb >= 0x1p62f);
        }
      }
      if (any_wave(large, 0)) {
        vm_wait_barrier<0>();
        return false;
      }
    }
#pragma unroll
    for (int u = 0; u < NP; ++u) split(f0, u);
    int g = 0;
    for (; g + 2 < steps; g += 2) {
      step(f0, f1, g + 1);
      step(f1, f0, g + 2);
    }
    if (g + 1 < steps) {
      step(f0, f1, g + 1);
      last(f1);
    } else {
      last(f0);
    }
    float nan = 0.f;   // becomes NaN when a sum is not finite
    bool redo = false;
    const int rows = (int)min(M - m0 - wm0, (int64_t)(32 * SUB)), cols = (int)min(N - n0 - wn0, (int64_t)(32 * SUB));
    // Rows and columns that are stored and hold no NaN (where one does, every
    // output is NaN in any arithmetic): of rows a mask, of columns the lane's own.
    uint32_t rows_in[SUB];
    bool col_in[SUB];
    float row_most[SUB], col_most[SUB];
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
      // both lane halves hold K positions of row / column r32
      row_most[i] = largest(most_a[i], __shfl_xor(most_a[i], 32));
      col_most[i] = largest(most_b[i], __shfl_xor(most_b[i], 32));
      col_in[i] = 32 * i + r32 < cols && col_most[i] == col_most[i];
      rows_in[i] = (uint32_t)__ballot(32 * i + r32 < rows && row_most[i] == row_most[i]) >> (4 * h);
    }
#pragma unroll
    for (int i = 0; i < SUB; ++i)
#pragma unroll
      for (int j = 0; j < SUB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool in = col_in[j] && (rows_in[i] >> ((r >> 2) * 8 + (r & 3)) & 1u) != 0u;
          nan = fmaf(in ? sacc[i][j][r] : 0.f, 0.f, nan);
        }
    if (__any((left & 0xffffu) != 0u)) {
      // what the pieces leave out of a sum is at most 2^-134 K (row_most + col_most)
      const float unit = (float)K * 0x1p-107f;
#pragma unroll
      for (int i = 0; i < SUB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = (r >> 2) * 8 + (r & 3);
          const float m = __shfl(row_most[i], row + 4 * h);
#pragma unroll
          for (int j = 0; j < SUB; ++j)
            redo = redo || (col_in[j] && (rows_in[i] >> row & 1u) != 0u && m > 0.f && col_most[j] > 0.f &&
                            !(__builtin_fabsf(sacc[i][j][r]) >= unit * (m + col_most[j])));
        }
    }
    return !any_wave(redo || nan != nan, 1);
  };
  // T = 2 carries its running sums to `total` every 256 of K: a chain of K / 4
  // rounded additions is what deep products lose most by (1021 x 515 x 997:
  // 5.6e-7 against 64 bits in one chain, 2.9e-7 in blocks).
  constexpr int SUM_STAGES = T == 2 ? 256 / BK : INT_MAX;
  start(wave, lane);
  bool done = false;
  int lane_f = lane, wave_f = wave;
  if constexpr (SPLIT) {
    done = split_product();
    // the second pass works out its addresses by itself: shared with the first
    // they would have to stay in registers through it
    asm volatile("" : "+v"(lane_f), "+s"(wave_f));
    if (!done) {
      clear();
      start(wave_f, lane_f);
    }
  }
  // The products of the stage held at `cur`.
  auto products = [&](const char* cur) __attribute__((always_inline)) {
    const float* as = reinterpret_cast<const float*>(cur);
    const float* bs = reinterpret_cast<const float*>(cur + Cfg::A_BYTES);
    if constexpr (T == 2) {
      // 16x16x4: lane quarter g = lane / 16 takes k = g * BK / 4 + q
      const int r16 = lane & 15, g = lane >> 4;
      constexpr int KQ = BK / 4;
      f32x4 c = {acc[0], acc[1], acc[2], acc[3]};
      // element reads, which the compiler merges where it can (explicit
      // 16-byte reads measured 3 % slower here on the mixed layouts); 64 deep,
      // all in flight before the first MFMA (left to the scheduler, each
      // MFMA group waited for its own: 1021x515x997 NT 54.6 -> 50.6 us, 4 x
      // 1x4096x6272 81 -> 75 us on (32, 32, 2, 64); 32 deep it gains nothing)
      float a[KQ], b[KQ];
#pragma unroll
      for (int q = 0; q < KQ; ++q) {
        a[q] = A_at(as, wm0 + r16, g * KQ + q);
        b[q] = B_at(bs, wn0 + r16, g * KQ + q);
      }
      if (BK >= 64) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < KQ; ++q) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], b[q], c, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = c[r];
    } else if constexpr (T == 4) {
      const int r32 = lane & 31, h = lane >> 5;
      constexpr int KH = BK / 2;
      f32x16 c;
#pragma unroll
      for (int r = 0; r < 16; ++r) c[r] = acc[r];
      static_assert(KH % 4 == 0, "whole 16-byte chunks per lane half");
#pragma unroll
      for (int q0 = 0; q0 < KH; q0 += 4) {
        const f32x4 a = A4(as, wm0 + r32, h * KH + q0);
        const f32x4 b = B4(bs, wn0 + r32, h * KH + q0);
#pragma unroll
        for (int u = 0; u < 4; ++u) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u], b[u], c, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = c[r];
    } else {
      const int r32 = lane_f & 31, h = lane_f >> 5;
      constexpr int KH = BK / 2;
      static_assert(KH % 4 == 0, "whole 16-byte chunks per lane half");
      auto group = [&](int k) __attribute__((always_inline)) {
        const int wm0 = (wave_f / Cfg::Base::WAVES_N) * WT, wn0 = (wave_f % Cfg::Base::WAVES_N) * WT;
        const f32x4 a0 = A4(as, wm0 + r32, k), a1 = A4(as, wm0 + 32 + r32, k);
        const f32x4 b0 = B4(bs, wn0 + r32, k), b1 = B4(bs, wn0 + 32 + r32, k);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          sacc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[u], b0[u], sacc[0][0], 0, 0, 0);
          sacc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[u], b1[u], sacc[0][1], 0, 0, 0);
          sacc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[u], b0[u], sacc[1][0], 0, 0, 0);
          sacc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[u], b1[u], sacc[1][1], 0, 0, 0);
        }
      };
#pragma unroll
      for (int q0 = 0; q0 < KH; q0 += 4) {
        if constexpr (SPLIT) __builtin_amdgcn_sched_barrier(0);   // no more registers than the first pass
        group(h * KH + q0);
      }
    }
  };
  const int lean = T == 8 || done ? 0 : src.lean_stages(nk);
  for (int kt = done ? nk : 0; kt < nk;) {
    const int end = T == 2 ? min(nk, kt + SUM_STAGES) : nk;
    if constexpr (T != 8) {
      for (const int to = min(end, lean); kt < to; ++kt) {
        lean_stage<Cfg>(src, kt, my_blocks == Cfg::NW_HI, lds0);
        products(lds + (uint32_t)kt % NS * Cfg::STAGE);
      }
    }
    for (; kt < end; ++kt) {
      open_stage(kt, kt + NS - 1, NS - 2);
      products(lds + (kt % NS) * Cfg::STAGE);
    }
    if constexpr (T == 2) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        total[r] += acc[r];
        acc[r] = 0.f;
      }
    }
  }

  float* __restrict__ Cg = args.C + bz * args.sC;
  const float alpha = args.alpha, beta = args.beta;
  const int64_t ldc = args.ldc;
  auto put = [&](int row, int col, float v) {
    const int64_t gi = m0 + wm0 + row, gj = n0 + wn0 + col;
    if (gi < M && gj < N) {
      float* p = Cg + gi * ldc + gj;
      float out = alpha * v;
      if (beta != 0.f) out = fmaf(beta, *p, out);
      *p = out;
    }
  };
  auto put_blocks = [&](const f32x16 (&c)[SUB][SUB]) {
#pragma unroll
    for (int i = 0; i < SUB; ++i)
#pragma unroll
      for (int j = 0; j < SUB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          put(32 * i + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), 32 * j + (lane & 31), c[i][j][r]);
  };
  if constexpr (T == 8) {
    put_blocks(sacc);
  } else if constexpr (T == 2) {
#pragma unroll
    for (int r = 0; r < 4; ++r) put((lane >> 4) * 4 + r, lane & 15, total[r]);
  } else if constexpr (T == 4) {
#pragma unroll
    for (int r = 0; r < 16; ++r) put((r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), lane & 31, acc[r]);
  }
}

// Configurations the DMA pipeline serves: the 16x16 and 32x32 MFMA families
// whose tiles are whole 1 KiB DMA blocks.
template <int BM, int BN, int T, int BK>
struct F32DmaServes {
  static constexpr bool value = T >= 2 && (BM * BK * 4) % 1024 == 0 && (BN * BK * 4) % 1024 == 0;
};

// Host-side launcher of one instantiation on a stream.  Operands whose rows
// start on 4-byte boundaries and hold at least one 16-byte chunk take the DMA
// pipeline where the configuration has one (the split kernels from K = 16:
// less deep products are more exact with FP32 MFMAs): global loads need
// dword alignment only, a chunk that runs over the end of its row reads into
// the next one, and only the chunk at the very end of an operand is moved
// (DmaSource::settle).  Any other operand takes the register-staged kernel.
// Dense 1001x1003x1005 NN: (32, 32, 2, 32) 37.5 -> 28.1 us, (64, 64, 4, 32)
// 45.9 -> 33.0 us, (128, 128, 8, 16) 134 -> 57 us (the last on the split kernel).
// Such rows need a K that fills the stages: a shallow product has no use for
// their LDS, which costs it resident work-groups, and its last stage takes a
// pass more.  8 x 500x500 dense: on (32, 32, 2, 64) register-staged / DMA 14.6 / 19.7
// us at K = 65, 18.8 / 23.0 at 129, 9.2 / 7.5 at 257 (4 x 250x251); on (64, 64, 4, 16)
// 7.8 / 8.0 at 33, 9.8 / 9.4 at 65, 13.9 / 12.2 at 129; on (128, 64, 4, 32) 10.1 /
// 10.2 at 65, 13.7 / 13.0 at 129.
template <int T, int BK>
struct F32DenseK {
  static constexpr int value = T == 2 ? 256 : 3 * BK;
};

template <int BM, int BN, int T, int BK, int TA, int TB>
hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t stream) {
  using Cfg = GemmF32Cfg<BM, BN, T, BK, TA, TB>;
  if constexpr (F32DmaServes<BM, BN, T, BK>::value) {
    if (a.alignA >= ROWS_4 && a.alignB >= ROWS_4 && a.K >= (F32Split<T, BK>::value ? 16 : 4) &&
        (TA == 0 || a.M >= 4) && (TB == 1 || a.N >= 4)) {
      GemmArgs g = a;
      g.ragged = a.alignA != ROWS_16 || a.alignB != ROWS_16;
      if (!g.ragged || a.K >= F32DenseK<T, BK>::value)
        return launch_flat<4>(gemm_f32_dma_kernel<BM, BN, T, BK, TA, TB>, g, BM, BN, Cfg::NT, stream);
    }
  }
  return launch_flat<4>(gemm_f32_kernel<BM, BN, T, BK, TA, TB>, a, BM, BN, Cfg::NT, stream);
}

}  // namespace kt
