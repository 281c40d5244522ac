// Direct-to-LDS pipeline of the low-precision family, taken when every
// operand row starts on a 16-byte boundary (base, leading dimension and
// batch stride multiples of 16 bytes) and no 16-byte chunk read can leave
// the operand: its contiguous extent (K, or M / N for an operand stored M- /
// N-contiguous) is whole chunks, or (grouped members, whose rows are
// allocated to the full leading dimension) the last chunk of a row ends
// within the leading dimension.  Same configuration knobs and results
// contract as gemm_lp.hpp; what changes is how tiles reach the MFMAs:
//
// * Global -> LDS with gfx950's 16-byte LDS DMA (global_load_lds_dwordx4):
//   each wave instruction moves 1 KiB straight into LDS (lane l's 16 bytes
//   land at the instruction's LDS base + 16 l), with no register staging, so
//   NS stages (2..4, as many as the LDS budget allows) are in flight at once
//   and a stage is waited for with vmcnt, not refetched through VGPRs.
// * An operand stored with K contiguous keeps that layout in LDS ([row][k],
//   rows of BK elements); its MFMA fragments are 16-byte LDS reads.  The
//   16-byte chunks of a row are XOR-swizzled by the row index so that the 16
//   rows one read phase touches fall on distinct bank groups.
// * An operand stored with M (or N) contiguous is copied as stored
//   ([k][col]) and its fragments come from the LDS transpose reads
//   (ds_read_b64_tr_b16 for BF16: lane j of a 16-lane group receives four
//   consecutive k of column j from the 4 x 16 block the group addresses;
//   ds_read_b64_tr_b8 for FP8: eight consecutive k of column j from an
//   8 x 16 block), chunks swizzled by k so the rows read together spread
//   over the banks.
// * Out-of-range rows and columns are read from clamped in-range addresses
//   (those outputs are never stored); K beyond the product in the last stage
//   is zeroed in LDS after it lands, so it adds nothing.
#pragma once
#include "gemm_lp.hpp"

namespace kt {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void gbl_void_t;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));

// LDS byte address of a pointer into a workgroup's shared array.
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)p);
}

// Wait until at most N of this wave's vector-memory operations (the LDS DMA
// of later stages) are outstanding and its LDS reads have returned, then
// meet the other waves.  One asm block, so nothing is moved across it.
template <int N>
__device__ __forceinline__ void vm_wait_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// One lane's 16 bytes of a wave's 1 KiB LDS DMA: global `src` to the LDS
// block at `dst` (wave-uniform; lane l's bytes land at dst + 16 l).  Written
// as inline asm so the compiler does not track it: its waitcnt pass cannot
// tell which stage buffer a transpose read touches and otherwise waits for
// every DMA in flight -- the next stage's included -- before each stage's
// fragment reads.  Every wait on these transfers is the explicit one of the
// stage pipeline (vm_wait_barrier); vector-memory operations complete in
// issue order, so the compiler's own vmcnt waits stay correct.
__device__ __forceinline__ void lds_dma16(const void* src, uint32_t m0) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "{m0}"(m0));
}

// The same with a wave-uniform base, a 32-bit byte offset per lane and the
// LDS address in a scalar.  The base is moved inside the block: a vector
// memory instruction may not read a scalar register within five wait states
// of a vector instruction's write (a readfirstlane, a spilled scalar read
// back with readlane), a hazard the compiler does not look for in inline asm;
// a scalar move waits for such a write by itself, and stands between the
// write of M0 and its use.
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t off, uint32_t m0) {
  uint64_t t;
  asm volatile("s_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
               : "=&s"(t)
               : "v"(off), "s"(base), "{m0}"(m0));
}

// A pointer whose value is the same in every lane, in scalar registers.
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const char*>((uintptr_t)(((uint64_t)hi << 32) | lo));
}

template <int EB, int BM, int BN, int T, int BK, int TA, int TB>
struct LpDmaCfg {
  using Base = GemmLpCfg<EB, BM, BN, T, BK, TA, TB>;
  static constexpr int NT = Base::NT, WAVES = Base::WAVES;
  static constexpr int A_BYTES = BM * BK * EB, B_BYTES = BN * BK * EB;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  // Large tiles run one work-group per CU and take as many stages as fit;
  // smaller ones leave room for a second work-group.
  static constexpr int BUDGET = (BM * BN >= 256 * 128) ? 160 * 1024 : 80 * 1024;
  static constexpr int NS_FIT = BUDGET / STAGE;
  static constexpr int NS = NS_FIT < 2 ? 2 : (NS_FIT > 4 ? 4 : NS_FIT);
  static constexpr int LDS_BYTES = NS * STAGE;
  static constexpr int NBA = A_BYTES / 1024, NBB = B_BYTES / 1024;   // 1 KiB DMA blocks
  static constexpr int NBLK = NBA + NBB;
  static constexpr int NW_LO = NBLK / WAVES, NW_HI = (NBLK + WAVES - 1) / WAVES;
  // Occupancy target: the waves per SIMD that the LDS footprint allows,
  // capped at 2, so the register budget (512 / waves) keeps a second
  // work-group resident wherever the LDS has room for it.
  static constexpr int OCC_LDS = (160 * 1024 / LDS_BYTES) * WAVES / 4;
  static constexpr int OCC = OCC_LDS < 1 ? 1 : (OCC_LDS > 2 ? 2 : OCC_LDS);
  static_assert(A_BYTES % 1024 == 0 && B_BYTES % 1024 == 0, "tiles of whole 1 KiB blocks");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
  static_assert((NS - 2) * NW_HI < 64, "vmcnt range");
};

// Stage wait: at most `ahead` (0 .. NS - 2) later stages of NW blocks each
// may still be in flight.
template <int NW, int NS>
__device__ __forceinline__ void wait_stage(int ahead) {
  if constexpr (NS >= 4) {
    if (ahead >= 2) { vm_wait_barrier<2 * NW>(); return; }
  }
  if constexpr (NS >= 3) {
    if (ahead >= 1) { vm_wait_barrier<NW>(); return; }
  }
  vm_wait_barrier<0>();
}

// The start of a stage whose successors are all under way (DmaSource::
// lean_stages): its DMA has landed for every wave, and the stage NS - 1 on is
// issued into the buffer that every wave has finished reading.  Of a K loop all
// stages but the last few are of this kind, and of them the short ones are bound
// by the one scalar unit of a CU: with the general test of the stage's place
// ((64, 64, 2, 8) in FP32, two work-groups of sixteen waves, 80 scalar
// instructions a wave and stage) a stage took 1.05 us, without it 0.55.
template <typename Cfg, typename Src>
__device__ __forceinline__ void lean_stage(Src& src, int kt, bool hi, uint32_t lds0) {
  constexpr int NS = Cfg::NS;
  if (Cfg::NW_HI == Cfg::NW_LO || hi) vm_wait_barrier<(NS - 2) * Cfg::NW_HI>();
  else vm_wait_barrier<(NS - 2) * Cfg::NW_LO>();
  src.issue_whole(lds0 + (uint32_t)(kt + NS - 1) % NS * Cfg::STAGE);
}

// Chunk swizzles.  K-major rows hold CPR 16-byte chunks; chunk c of row r
// sits at c ^ kswz(r): the 16 consecutive rows a fragment read touches land
// on 16 distinct 16-byte bank groups of the 256-byte bank line.
template <int CPR>
__device__ __forceinline__ int kswz(int r) {
  constexpr int RP = CPR >= 16 ? 1 : 16 / CPR;   // rows per 256 bytes
  return (r / RP) % CPR;
}
// MN-major rows (one k each): the rows a transpose read covers together
// (4 for BF16, 8 for FP8, each W = 16 / rows chunks wide) are moved W chunks
// apart per 256-byte line.
template <int CPR, int W>
__device__ __forceinline__ int mswz(int k) {
  constexpr int RP = CPR >= 16 ? 1 : 16 / CPR;
  return ((k / RP) * W) % CPR;
}

// A lane's value for work that a loop seldom does: what follows from it is
// worked out there, not ahead of the loop in registers that the loop needs.
// FP32 kernels only: low-precision ones have no branches that need it, and
// BF16 NN on (256, 256, 8, 64) spilled with it.
__device__ __forceinline__ int rarely(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Where a wave's DMA blocks of one stage come from.  Block q of the stage
// (0 .. NBA-1: A, then B) is handled by wave q % WAVES; rows / columns beyond
// the operand are clamped to in-range addresses.
//
// Every stage reads the same places relative to its first k, so each lane's
// 32-bit offset of each block is computed once and a stage costs one scalar
// base per operand and one move per block.  Recomputed per stage (64-bit
// row * ld + k with clamps, 15 to 25 vector instructions a block) the
// addresses competed with the MFMAs for issue slots and, in the grouped
// kernel, for registers: 512 BF16 members 651 -> 441 us, BF16 4096^3 with its
// conversion 174 -> 164 us, FP32 4096^3 NN 1080 -> 1017 us.  The last, partial
// stage moves the offsets beyond K back to the last chunk or row; operands
// whose tile spans 2^31 bytes or more (ld >= 2^31 / (tile rows * EB): the
// offsets would not hold) compute whole addresses.
template <typename Cfg, int EB, int BM, int BN, int BK, int TA, int TB, typename Swz>
struct DmaSource {
  static constexpr int CE = 16 / EB;   // elements per chunk
  uint32_t off[Cfg::NW_HI];
  const char* a;                       // first element of the tile at the next stage's first k
  const char* b;
  int64_t step_a, step_b;              // bytes per stage
  int wave, lane;
  int whole;                           // whole stages left to issue
  int tail;                            // K positions of the stage after them
  bool offsets;                        // the 32-bit offsets hold
  bool ragged;                         // rows on 4-byte boundaries only (GemmArgs::ragged)

  // Chunk of block q this lane moves: tile row (K-major) or k (M/N-major)
  // and element column.
  __device__ __forceinline__ static void place(int q, int lane, bool& is_a, bool& kmajor, int& r,
                                               int& col) {
    is_a = q < Cfg::NBA;
    const int o = (is_a ? q : q - Cfg::NBA) * 1024 + lane * 16;   // byte in the operand's tile
    kmajor = is_a ? (TA == 0) : (TB == 1);
    if (kmajor) {
      constexpr int ROWB = BK * EB;
      r = o / ROWB;
      col = (((o % ROWB) / 16) ^ Swz::k(r)) * CE;
    } else {
      const int rowb = (is_a ? BM : BN) * EB;
      r = o / rowb;
      col = (((o % rowb) / 16) ^ (is_a ? Swz::mn_a(r) : Swz::mn_b(r))) * CE;
    }
  }

  __device__ __forceinline__ static int seldom(int v) { return EB == 4 ? rarely(v) : v; }

  // Whether block i of every wave exists, and whether it is one of A's for
  // every wave / for none; only where the blocks do not divide evenly is
  // either asked of the wave.
  __device__ __forceinline__ bool exists(int i) const {
    return (i + 1) * Cfg::WAVES <= Cfg::NBLK || wave + i * Cfg::WAVES < Cfg::NBLK;
  }
  __device__ __forceinline__ bool of_a(int i) const {
    if ((i + 1) * Cfg::WAVES <= Cfg::NBA) return true;
    return i * Cfg::WAVES < Cfg::NBA && wave + i * Cfg::WAVES < Cfg::NBA;
  }

  // Offsets of block i beyond K in the last stage, which holds left_k of it, moved
  // back to its last chunk or row.
  __device__ __forceinline__ uint32_t in_tail(const GemmArgs& g, int i, int left_k, int lane) const {
    bool is_a, kmajor;
    int r, col;
    place(wave + i * Cfg::WAVES, lane, is_a, kmajor, r, col);
    if (kmajor) return off[i] - (uint32_t)max(col - (left_k - 1) / CE * CE, 0) * EB;
    return off[i] - (uint32_t)max(r - (left_k - 1), 0) * (uint32_t)((is_a ? g.lda : g.ldb) * EB);
  }

  __device__ __forceinline__ void init(const GemmArgs& g, const char* Ag, const char* Bg,
                                       int64_t m0, int64_t n0, int wave_, int lane_) {
    wave = wave_;
    lane = lane_;
    a = uniform_ptr(Ag + m0 * (TA == 0 ? g.lda : 1) * EB);
    b = uniform_ptr(Bg + n0 * (TB == 1 ? g.ldb : 1) * EB);
    step_a = (int64_t)BK * (TA == 0 ? 1 : g.lda) * EB;
    step_b = (int64_t)BK * (TB == 1 ? 1 : g.ldb) * EB;
    whole = (int)((uint64_t)g.K / BK);
    tail = (int)((uint64_t)g.K % BK);
    // tile rows times ld below 2^31 bytes (shifts: compares of 64-bit values
    // leave the scalar unit)
    constexpr int LOG_A = 31 - __builtin_ctz((TA == 0 ? BM : BK) * EB);
    constexpr int LOG_B = 31 - __builtin_ctz((TB == 1 ? BN : BK) * EB);
    offsets = (((uint64_t)g.lda >> LOG_A) | ((uint64_t)g.ldb >> LOG_B)) == 0;
    ragged = EB == 4 && g.ragged != 0;
    const uint64_t over_m = (uint64_t)(g.M - m0), over_n = (uint64_t)(g.N - n0);
    const int left_m = (over_m >> 31) ? BM : min(BM, (int)over_m);
    const int left_n = (over_n >> 31) ? BN : min(BN, (int)over_n);
#pragma unroll
    for (int i = 0; i < Cfg::NW_HI; ++i) {
      bool is_a, kmajor;
      int r, col;
      place(exists(i) ? wave + i * Cfg::WAVES : 0, lane, is_a, kmajor, r, col);
      const int left = is_a ? left_m : left_n;   // rows or columns
      const uint32_t ld = (uint32_t)(is_a ? g.lda : g.ldb);
      if (kmajor) r = min(r, left - 1);
      else col = min(col, (int)((uint32_t)(left - 1) / CE * CE));
      off[i] = ((uint32_t)r * ld + (uint32_t)col) * EB;
    }
  }

  // Offsets, in the last stage, of the last 16 bytes of A and B where the tile
  // holds them: the only chunk of the operand that starts later is the one that
  // runs over its end.  False when they start before the tile.
  __device__ __forceinline__ bool ends(const GemmArgs& g, int64_t m0, int64_t n0, int left_k,
                                       uint32_t& ea, uint32_t& eb) const {
    const uint64_t over_m = (uint64_t)(g.M - m0), over_n = (uint64_t)(g.N - n0);
    const int left_m = (over_m >> 31) ? BM + 1 : min(BM + 1, (int)over_m);
    const int left_n = (over_n >> 31) ? BN + 1 : min(BN + 1, (int)over_n);
    const int lda = (int)g.lda, ldb = (int)g.ldb;
    const int la = (TA == 0 ? (left_m - 1) * lda + left_k : (left_k - 1) * lda + left_m) - CE;
    const int lb = (TB == 1 ? (left_n - 1) * ldb + left_k : (left_k - 1) * ldb + left_n) - CE;
    ea = left_m <= BM ? (uint32_t)la * EB : ~0u;
    eb = left_n <= BN ? (uint32_t)lb * EB : ~0u;
    return (left_m > BM || la >= 0) && (left_n > BN || lb >= 0);
  }

  // Stages whose successor NS - 1 stages on may be issued by issue_whole: it is
  // whole and not the last, and the offsets hold.
  __device__ __forceinline__ int lean_stages(int nk) const { return offsets ? nk - Cfg::NS : 0; }

  // Issue such a stage into the LDS at byte address `stage`.
  __device__ __forceinline__ void issue_whole(uint32_t stage) {
#pragma unroll
    for (int i = 0; i < Cfg::NW_HI; ++i)
      if (exists(i))
        lds_dma16(of_a(i) ? a : b, off[i], stage + (wave + i * Cfg::WAVES) * 1024);
    a += step_a;
    b += step_b;
    --whole;
  }

  // Issue the next stage, any, into the LDS at byte address `stage`.
  __device__ __forceinline__ void issue(const GemmArgs& g, int64_t m0, int64_t n0, uint32_t stage) {
    const bool last = whole <= (tail == 0 ? 1 : 0), end = ragged && last;
    const int left_k = whole > 0 ? BK : tail;
    uint32_t ea = ~0u, eb = ~0u;
    if (offsets && (!end || ends(g, m0, n0, left_k, ea, eb))) {
      if (whole > 0 && !end) {
#pragma unroll
        for (int i = 0; i < Cfg::NW_HI; ++i)
          if (exists(i))
            lds_dma16(of_a(i) ? a : b, off[i], stage + (wave + i * Cfg::WAVES) * 1024);
      } else {
        const int l = seldom(lane);
#pragma unroll
        for (int i = 0; i < Cfg::NW_HI; ++i)
          if (exists(i))
            lds_dma16(of_a(i) ? a : b,
                      EB == 4 ? min(in_tail(g, i, left_k, l), of_a(i) ? ea : eb) : in_tail(g, i, left_k, l),
                      stage + (wave + i * Cfg::WAVES) * 1024);
      }
    } else {
      // whole addresses: a loop, out of the way of the products that have offsets
      const int l = seldom(lane);
#pragma nounroll
      for (int q = wave; q < Cfg::NBLK; q += Cfg::WAVES) {
        bool is_a, kmajor;
        int r, col;
        place(q, l, is_a, kmajor, r, col);
        const int64_t left = is_a ? g.M - m0 : g.N - n0;
        const int64_t ld = is_a ? g.lda : g.ldb;
        int64_t row = r, c = col;
        if (kmajor) {
          row = min(row, left - 1);
          c = min(col, (left_k - 1) / CE * CE);       // chunks beyond K: the last one
          if (ragged && last && row == left - 1) c = min(c, (int64_t)left_k - CE);
        } else {
          row = min(r, left_k - 1);
          c = min(c, (left - 1) / CE * CE);           // chunks beyond the extent: the last one
          if (ragged && last && row == left_k - 1) c = min(c, left - CE);
        }
        lds_dma16((is_a ? a : b) + (row * ld + c) * EB, stage + q * 1024);
      }
    }
    a += step_a;
    b += step_b;
    --whole;
  }

  // The chunk at the very end of a ragged operand was read so that it ends
  // with the operand (every other chunk that runs over its row's extent stays
  // inside the next row); move its values to their places.  Called for the
  // last stage, landed, by every thread; true when a barrier is needed after.
  __device__ __forceinline__ bool settle(const GemmArgs& g, int64_t m0, int64_t n0, int left_k,
                                         char* stage, int tid) const {
    if (!ragged) return false;
    tid = rarely(tid);
    if (tid < 2) {   // one thread per operand
      const bool is_a = tid == 0, kmajor = is_a ? (TA == 0) : (TB == 1);
      const int64_t left = is_a ? g.M - m0 : g.N - n0;
      const int rows = is_a ? BM : BN;
      if (left <= rows) {   // the tile that holds the operand's last row or column
        const int ext = kmajor ? left_k : (int)left;
        const int c = (ext - 1) / CE * CE, shift = c + CE - ext;
        const int r = kmajor ? (int)left - 1 : left_k - 1;
        const int sw = kmajor ? Swz::k(r) : is_a ? Swz::mn_a(r) : Swz::mn_b(r);
        float* p = reinterpret_cast<float*>(stage + (is_a ? 0 : Cfg::A_BYTES)) +
                   r * (kmajor ? BK : rows) + ((c / CE) ^ sw) * CE;
        for (int e = 0; e + shift < CE; ++e) p[e] = p[e + shift];
      }
    }
    return true;
  }
};

template <int EB, int BM, int BN, int BK>
struct LpSwz {
  __device__ __forceinline__ static int k(int r) { return kswz<BK * EB / 16>(r); }
  __device__ __forceinline__ static int mn_a(int r) { return mswz<BM * EB / 16, EB == 2 ? 4 : 2>(r); }
  __device__ __forceinline__ static int mn_b(int r) { return mswz<BN * EB / 16, EB == 2 ? 4 : 2>(r); }
};

// Zero K positions kvalid .. BK-1 of a stage (the last, partial one).
template <int EB, int BM, int BN, int T, int BK, int TA, int TB>
__device__ __forceinline__ void lp_dma_zero_tail(char* stage, int kvalid, int tid) {
  using Cfg = LpDmaCfg<EB, BM, BN, T, BK, TA, TB>;
  typedef typename LpElem<EB>::T E;
  asm volatile("" : "+s"(kvalid));   // keeps this rarely run arithmetic out of the stage loop's preheader
#pragma unroll
  for (int op = 0; op < 2; ++op) {
    const bool kmajor = op == 0 ? (TA == 0) : (TB == 1);
    const int rows_c = op == 0 ? BM : BN;
    E* t = reinterpret_cast<E*>(stage + (op == 0 ? 0 : Cfg::A_BYTES));
    if (kmajor) {
      constexpr int CPR = BK * EB / 16, CE = 16 / EB;
      for (int i = tid; i < rows_c * CPR; i += Cfg::NT) {
        const int r = i / CPR, c = i % CPR;
        E* p = t + r * BK + (c ^ kswz<CPR>(r)) * CE;
        const int from = kvalid - CE * c;   // first element to clear
        if (from <= 0) *reinterpret_cast<u32x4*>(p) = u32x4{0u, 0u, 0u, 0u};
        else
          for (int e = from; e < CE; ++e) p[e] = (E)0;
      }
    } else {
      const int per = rows_c * EB / 16;   // chunks per row
      for (int i = kvalid * per + tid; i < BK * per; i += Cfg::NT)
        reinterpret_cast<u32x4*>(t)[i] = u32x4{0u, 0u, 0u, 0u};
    }
  }
}

// One lane's MFMA fragment of MFMA block `blk` (rows or columns blk * MB ..)
// for K step s of a stage tile held K-major.
template <int EB, int BK, int MB, int KSTEP>
__device__ __forceinline__ void lp_frag_kmajor(LpFrag<EB>& f, const char* tile, int row, int s,
                                               int kh) {
  constexpr int CPR = BK * EB / 16;
  const int c = (s * KSTEP + kh) * EB / 16;
  const char* rp = tile + row * (BK * EB);
  if constexpr (EB == 2) {
    f.v = *reinterpret_cast<const bf16x8*>(rp + (c ^ kswz<CPR>(row)) * 16);
  } else {
    const u32x4 lo = *reinterpret_cast<const u32x4*>(rp + (c ^ kswz<CPR>(row)) * 16);
    const u32x4 hi = *reinterpret_cast<const u32x4*>(rp + ((c + 1) ^ kswz<CPR>(row)) * 16);
    i32x8 v;
    v[0] = lo[0]; v[1] = lo[1]; v[2] = lo[2]; v[3] = lo[3];
    v[4] = hi[0]; v[5] = hi[1]; v[6] = hi[2]; v[7] = hi[3];
    f.v = v;
  }
}

// The same for a tile held MN-major ([k][col], COLS columns): transpose
// reads.  colg is the first column of this lane's 16-lane group, kg its
// first k in the stage.
template <int EB, int COLS>
__device__ __forceinline__ void lp_frag_mnmajor(LpFrag<EB>& f, const char* tile, int colg, int kg,
                                                int j) {
  constexpr int ROWB = COLS * EB, CPR = ROWB / 16;
  if constexpr (EB == 2) {
    // source lane j = 4 r + c reads k row kg + kq + r, columns colg + 4c .. + 3
    const int r = j >> 2, cq = j & 3;
    const int byte = (colg + 4 * cq) * 2;
    s16x4 h[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int k = kg + 4 * q + r;
      const char* p = tile + k * ROWB + (((byte >> 4) ^ mswz<CPR, 4>(k)) << 4) + (byte & 15);
      h[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
    }
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    s16x8 v;
    v[0] = h[0][0]; v[1] = h[0][1]; v[2] = h[0][2]; v[3] = h[0][3];
    v[4] = h[1][0]; v[5] = h[1][1]; v[6] = h[1][2]; v[7] = h[1][3];
    f.v = __builtin_bit_cast(bf16x8, v);
  } else {
    // source lane j = 2 r + c reads k row kg + 8q + r, columns colg + 8c .. + 7
    const int r = j >> 1, cq = j & 1;
    const int byte = colg + 8 * cq;
    i32x8 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = kg + 8 * q + r;
      const char* p = tile + k * ROWB + (((byte >> 4) ^ mswz<CPR, 2>(k)) << 4) + (byte & 15);
      const i32x2 w = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i32x2*)(p));
      v[2 * q] = w[0];
      v[2 * q + 1] = w[1];
    }
    f.v = v;
  }
}

// What both pipelines of a tile share: a wave's accumulators, the products of
// one stage in LDS, and the epilogue.
template <int EB, int BM, int BN, int T, int BK, int TA, int TB>
struct LpTileMath {
  using Cfg = LpDmaCfg<EB, BM, BN, T, BK, TA, TB>;
  using Base = typename Cfg::Base;
  static constexpr int WT = Base::WT, MB = Base::MB, SUB = Base::SUB, KSTEP = Base::KSTEP;
  static constexpr int NACC = MB == 16 ? 4 : 16;
  typedef typename std::conditional<MB == 16, f32x4, f32x16>::type Acc;
  Acc acc[SUB][SUB];
  int lane, wm0, wn0;

  __device__ __forceinline__ void init(int wave, int l) {
    lane = l;
    wm0 = (wave / Base::WAVES_N) * WT;
    wn0 = (wave % Base::WAVES_N) * WT;
#pragma unroll
    for (int i = 0; i < SUB; ++i)
#pragma unroll
      for (int j = 0; j < SUB; ++j)
#pragma unroll
        for (int r = 0; r < NACC; ++r) acc[i][j][r] = 0.f;
  }

  __device__ __forceinline__ void stage(const char* at) {
    // lane l feeds row l % MB of its block with K values from group l / MB
    const int rb = lane % MB, kh = (lane / MB) * (KSTEP * MB / 64);
    const int j16 = lane & 15;
    const int gcol = rb - j16;   // first column of this lane's 16-lane group within its block
    const char* bt = at + Cfg::A_BYTES;
#pragma unroll
    for (int s = 0; s < BK / KSTEP; ++s) {
      LpFrag<EB> fa[SUB], fb[SUB];
#pragma unroll
      for (int i = 0; i < SUB; ++i) {
        if (TA == 0) lp_frag_kmajor<EB, BK, MB, KSTEP>(fa[i], at, wm0 + MB * i + rb, s, kh);
        else lp_frag_mnmajor<EB, BM>(fa[i], at, wm0 + MB * i + gcol, s * KSTEP + kh, j16);
        if (TB == 1) lp_frag_kmajor<EB, BK, MB, KSTEP>(fb[i], bt, wn0 + MB * i + rb, s, kh);
        else lp_frag_mnmajor<EB, BN>(fb[i], bt, wn0 + MB * i + gcol, s * KSTEP + kh, j16);
      }
#pragma unroll
      for (int i = 0; i < SUB; ++i)
#pragma unroll
        for (int j = 0; j < SUB; ++j) lp_mfma(fa[i], fb[j], acc[i][j]);
    }
  }

  __device__ __forceinline__ void store(const GemmArgs& args, int64_t m0, int64_t n0, int64_t bz,
                                        float scale) const {
    float* __restrict__ Cg = args.C + bz * args.sC;
    const float beta = args.beta;
#pragma unroll
    for (int i = 0; i < SUB; ++i)
#pragma unroll
      for (int j = 0; j < SUB; ++j)
#pragma unroll
        for (int r = 0; r < NACC; ++r) {
          // 32x32 blocks: row (r / 4) * 8 + (lane / 32) * 4 + r % 4; 16x16
          // blocks: row (lane / 16) * 4 + r; the column is lane % MB
          const int br = MB == 16 ? (lane >> 4) * 4 + r : (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
          const int64_t gi = m0 + wm0 + MB * i + br;
          const int64_t gj = n0 + wn0 + MB * j + lane % MB;
          if (gi < args.M && gj < args.N) {
            float* p = Cg + gi * args.ldc + gj;
            float out = scale * acc[i][j][r];
            if (beta != 0.f) out = fmaf(beta, *p, out);
            *p = out;
          }
        }
  }
};

// One BM x BN output tile through the DMA pipeline.  lds holds NS stages;
// the caller synchronizes before reusing it for another tile.
template <int EB, int BM, int BN, int T, int BK, int TA, int TB>
__device__ __forceinline__ void lp_dma_tile(const GemmArgs& args, int tm, int tn, int64_t bz,
                                            char* lds) {
  using Cfg = LpDmaCfg<EB, BM, BN, T, BK, TA, TB>;
  constexpr int NS = Cfg::NS;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = Cfg::WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lds0 = lds_address(lds);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int64_t K = args.K;
  DmaSource<Cfg, EB, BM, BN, BK, TA, TB, LpSwz<EB, BM, BN, BK>> src;
  src.init(args, static_cast<const char*>(args.A) + bz * args.sA * EB,
           static_cast<const char*>(args.B) + bz * args.sB * EB, m0, n0, wave, lane);
  float scale = args.alpha;
  if (EB == 1) scale = args.alpha / (args.scaleA[0] * args.scaleB[0]);

  LpTileMath<EB, BM, BN, T, BK, TA, TB> math;
  math.init(wave, lane);
  const int nk = (int)((K + BK - 1) / BK);
  const int my_blocks = (wave < Cfg::NBLK % Cfg::WAVES || Cfg::NBLK % Cfg::WAVES == 0)
                            ? Cfg::NW_HI : Cfg::NW_LO;

#pragma nounroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) src.issue(args, m0, n0, lds0 + s * Cfg::STAGE);

  int kt = 0;
  if constexpr (T == 2) {   // short stages; wider wave tiles have no use for a second loop
    for (const int lean = src.lean_stages(nk); kt < lean; ++kt) {
      lean_stage<Cfg>(src, kt, my_blocks == Cfg::NW_HI, lds0);
      math.stage(lds + (uint32_t)kt % NS * Cfg::STAGE);
    }
  }
  for (; kt < nk; ++kt) {
    // stage kt has landed once at most `ahead` later stages are in flight
    const int ahead = min(NS - 2, nk - 1 - kt);
    if (my_blocks == Cfg::NW_HI) wait_stage<Cfg::NW_HI, NS>(ahead);
    else wait_stage<Cfg::NW_LO, NS>(ahead);
    char* cur = lds + (kt % NS) * Cfg::STAGE;
    if (kt == nk - 1 && K - (int64_t)kt * BK < BK) {
      lp_dma_zero_tail<EB, BM, BN, T, BK, TA, TB>(cur, (int)(K - (int64_t)kt * BK), tid);
      vm_wait_barrier<0>();
    }
    // the buffer of stage kt - 1 is free: every wave has passed its reads
    if (kt + NS - 1 < nk)
      src.issue(args, m0, n0, lds0 + ((kt + NS - 1) % NS) * Cfg::STAGE);
    math.stage(cur);
  }
  math.store(args, m0, n0, bz, scale);
}

// Register staging of one operand of a tile into the layouts above, for
// operands that the DMA may not read: rows of any alignment.  A tile is ROWS
// rows of COLS contiguous elements (KM: rows of op's M or N, K contiguous;
// otherwise rows of K) in 16-byte chunks, chunk column tid % CPR of rows
// tid / CPR + i * STEP per thread.  A chunk is one 16-byte load from wherever
// it starts.  Rows beyond the operand repeat its last one and columns beyond
// it hold anything (those outputs are never stored): the chunk that straddles
// the last column is read so that it ends there, and shifted on its way to LDS.
// K beyond the product is zero.
// What bounds these tiles is the latency of a stage (loads, LDS stores,
// barrier), so their cost per load counts: with the transposition in registers
// that K-major LDS tiles need, and two loads per misaligned chunk, dense 8 x
// 1021x771x515 took 40.3 us in BF16 on (256, 128, 8, 64) and 41.4 in FP8, this
// way 25.5 and 20.3; 1023x1025x2047 76.8 and 51.0, this way 35.1 and 29.5; over all
// configurations of ten such products 1.8 times faster.
template <int EB, int ROWS, int COLS, bool KM, int NT>
struct StagedOperand {
  static constexpr int CE = 16 / EB, CPR = COLS / CE, NV = ROWS * CPR;
  static constexpr int PT = (NV + NT - 1) / NT, STEP = NT / CPR;
  static_assert(NT % CPR == 0, "one chunk column per thread");
  typedef uint32_t Chunk __attribute__((ext_vector_type(4), aligned(1)));
  const char* base;     // the tile's rows at the next stage's first k (uniform)
  int64_t ld;           // bytes
  uint32_t off[PT];
  int left;             // rows (KM) or columns of the operand from the tile's start
  int row0, col;        // this thread's first row, chunk column in elements
  bool plain, edge;     // 32-bit offsets and whole chunks; columns end inside the tile
  bool late;            // the chunks held wait for their shift
  u32x4 v[PT];

  __device__ __forceinline__ void init(const char* p, int64_t lde, int64_t first, int64_t ext, int tid) {
    ld = lde * EB;
    base = p + first * (KM ? ld : EB);
    const int64_t rem = ext - first;
    left = (int)min(rem, (int64_t)(KM ? ROWS : COLS));
    row0 = tid / CPR;
    col = (tid % CPR) * CE;
    edge = !KM && left < COLS;
    plain = (uint64_t)ld < (0x80000000ull / ROWS) && left >= (KM ? 1 : CE);
    const int c = edge ? min(col, left - CE) : col;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int r = row0 + i * STEP;
      off[i] = (uint32_t)(KM ? min(r, left - 1) : r) * (uint32_t)ld + (uint32_t)(c * EB);
    }
  }

  // Any chunk: elements one by one where the operand or K ends inside it.
  __device__ __forceinline__ u32x4 chunk(int row, int left_k) const {
    const int ext = KM ? left_k : row < left_k ? left : 0;
    const int n = min(ext - col, CE);
    const char* p = base + (KM ? min(row, left - 1) : row) * ld + col * EB;
    if (n == CE) return *reinterpret_cast<const Chunk*>(p);
    u32x4 t = {0u, 0u, 0u, 0u};
    if (n > 0) {
      typedef typename LpElem<EB>::T E;
#pragma unroll
      for (int e = 0; e < CE; ++e) {
        uint32_t x = 0u;
        __builtin_memcpy(&x, p + min(e, n - 1) * EB, EB);
        t[e * EB / 4] |= (e < n ? x : 0u) << (8 * (e * EB % 4));
      }
    }
    return t;
  }

  // Chunks of the next stage, which holds left_k of K.
  __device__ __forceinline__ void load(int64_t left_k) {
    const bool whole = plain && left_k >= (KM ? COLS : ROWS);
    late = whole && edge;
    if (whole) {
#pragma unroll
      for (int i = 0; i < PT; ++i)
        if (NV % NT == 0 || (int)threadIdx.x + i * NT < NV)
          v[i] = *reinterpret_cast<const Chunk*>(base + off[i]);
    } else {
      const int k = (int)min(left_k, (int64_t)(KM ? COLS : ROWS));
#pragma unroll
      for (int i = 0; i < PT; ++i)
        if (NV % NT == 0 || (int)threadIdx.x + i * NT < NV) v[i] = chunk(row0 + i * STEP, k);
    }
    base += KM ? COLS * EB : ROWS * ld;
  }

  // Chunks i0 .. i0 + G - 1 of the next stage, and their way to LDS; after all
  // of them, on to the stage behind it.
  template <int G>
  __device__ __forceinline__ void fetch(int i0, int64_t left_k, u32x4 (&t)[G]) const {
    const bool whole = plain && left_k >= (KM ? COLS : ROWS);
    const int k = (int)min(left_k, (int64_t)(KM ? COLS : ROWS));
    const uint32_t c = (uint32_t)(edge ? min(col, left - CE) : col) * EB;
    const int first = rarely(row0);   // no addresses kept from stage to stage
    if (whole) {
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int r = first + (i0 + u) * STEP;
        if (NV % (NT * G) == 0 || r < ROWS)
          t[u] = *reinterpret_cast<const Chunk*>(base + ((uint32_t)(KM ? min(r, left - 1) : r) * (uint32_t)ld + c));
      }
    } else {
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int r = first + (i0 + u) * STEP;
        if (NV % (NT * G) == 0 || r < ROWS) t[u] = chunk(r, k);
        __builtin_amdgcn_sched_barrier(0);   // one chunk's elements at a time
      }
    }
  }
  template <int G>
  __device__ __forceinline__ void place(int i0, int64_t left_k, u32x4 (&t)[G], char* tile) const {
    typedef unsigned __int128 u128;
    const bool shift = plain && edge && left_k >= ROWS;
    const int sh = shift ? min(max(col + CE - left, 0) * EB, 15) * 8 : 0;
    const int first = rarely(row0);
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int r = first + (i0 + u) * STEP;
      if (NV % (NT * G) == 0 || r < ROWS) {
        if (!KM && shift) t[u] = __builtin_bit_cast(u32x4, __builtin_bit_cast(u128, t[u]) >> sh);
        const int sw = KM ? kswz<CPR>(r) : mswz<CPR, EB == 2 ? 4 : 2>(r);
        *reinterpret_cast<u32x4*>(tile + r * (COLS * EB) + ((col / CE) ^ sw) * 16) = t[u];
      }
    }
  }
  template <int G>
  __device__ __forceinline__ void rest(int64_t left_k, u32x4 (&t)[G], char* tile) {
    place(0, left_k, t, tile);
#pragma nounroll
    for (int i0 = G; i0 < PT; i0 += G) {
      fetch(i0, left_k, t);
      place(i0, left_k, t, tile);
    }
    base += KM ? COLS * EB : ROWS * ld;
  }

  __device__ __forceinline__ void store(char* tile) {
    if (late) {
      const int sh = min(max(col + CE - left, 0) * EB, 15) * 8;
#pragma unroll
      for (int i = 0; i < PT; ++i) {
        typedef unsigned __int128 u128;
        v[i] = __builtin_bit_cast(u32x4, __builtin_bit_cast(u128, v[i]) >> sh);
      }
    }
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int r = row0 + i * STEP;
      const int sw = KM ? kswz<CPR>(r) : mswz<CPR, EB == 2 ? 4 : 2>(r);
      if (NV % NT == 0 || (int)threadIdx.x + i * NT < NV)
        *reinterpret_cast<u32x4*>(tile + r * (COLS * EB) + ((col / CE) ^ sw) * 16) = v[i];
    }
  }
};

// One BM x BN output tile with register-staged operands: the next stage's
// loads are in flight under the current stage's products, two stages in LDS.
template <int EB, int BM, int BN, int T, int BK, int TA, int TB>
__device__ __forceinline__ void lp_tile(const GemmArgs& args, int tm, int tn, int64_t bz, char* lds) {
  using Cfg = LpDmaCfg<EB, BM, BN, T, BK, TA, TB>;
  constexpr int NT = Cfg::NT;
  const int tid = threadIdx.x;
  const int wave = Cfg::WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int64_t K = args.K;
  StagedOperand<EB, TA == 0 ? BM : BK, TA == 0 ? BK : BM, TA == 0, NT> a;
  StagedOperand<EB, TB == 1 ? BN : BK, TB == 1 ? BK : BN, TB == 1, NT> b;
  a.init(static_cast<const char*>(args.A) + bz * args.sA * EB, args.lda, m0, args.M, tid);
  b.init(static_cast<const char*>(args.B) + bz * args.sB * EB, args.ldb, n0, args.N, tid);
  // FP8 per-tensor scales: loaded before the K loop so their latency is hidden
  float scale = args.alpha;
  if (EB == 1) scale = args.alpha / (args.scaleA[0] * args.scaleB[0]);
  LpTileMath<EB, BM, BN, T, BK, TA, TB> math;
  math.init(wave, tid & 63);
  const int nk = (int)((K + BK - 1) / BK);
  if constexpr (T == 16 && decltype(a)::PT + decltype(b)::PT >= 16) {
    // 256 accumulators a lane leave room for at most 15 chunks under the products
    // (16 and more: up to 2.7 KB of scratch memory a lane): these follow them,
    // eight of each operand in flight.  Dense 8 x 1021x771x515 NN in BF16, (128,
    // 256, 16, 64): 268 -> 105 us; (256, 256, 16, 32), 8 chunks: 80 us under the
    // products, 177 after them.
    for (int kt = -1; kt < nk; ++kt) {
      const int64_t left_k = K - (int64_t)(kt + 1) * BK;
      if (kt >= 0) math.stage(lds + (kt & 1) * Cfg::STAGE);
      __builtin_amdgcn_sched_barrier(0);
      if (left_k > 0) {
        char* next = lds + ((kt + 1) & 1) * Cfg::STAGE;
        u32x4 ta[8], tb[8];
        a.fetch(0, left_k, ta);
        b.fetch(0, left_k, tb);
        a.rest(left_k, ta, next);
        b.rest(left_k, tb, next + Cfg::A_BYTES);
      }
      __syncthreads();
    }
    math.store(args, m0, n0, bz, scale);
    return;
  }
  for (int kt = -1; kt < nk; ++kt) {   // -1: the first stage's loads
    const int64_t left_k = K - (int64_t)(kt + 1) * BK;
    if (left_k > 0) {
      a.load(left_k);
      b.load(left_k);
    }
    if (kt >= 0) math.stage(lds + (kt & 1) * Cfg::STAGE);
    if (left_k > 0) {
      char* next = lds + ((kt + 1) & 1) * Cfg::STAGE;
      a.store(next);
      b.store(next + Cfg::A_BYTES);
    }
    __syncthreads();
  }
  math.store(args, m0, n0, bz, scale);
}

template <int EB, int BM, int BN, int T, int BK, int TA, int TB>
__global__ void __launch_bounds__(BM * BN / (T * T))
__attribute__((amdgpu_waves_per_eu(LpDmaCfg<EB, BM, BN, T, BK, TA, TB>::OCC, 8)))
gemm_lp_kernel(GemmArgs args) {
  __shared__ __attribute__((aligned(16))) char lds[2 * LpDmaCfg<EB, BM, BN, T, BK, TA, TB>::STAGE];
  int tm, tn;
  int64_t bz;
  load_args(args);
  block_coords(blockIdx.x, args, tm, tn, bz);
  lp_tile<EB, BM, BN, T, BK, TA, TB>(args, tm, tn, bz, lds);
}

template <int EB, int BM, int BN, int T, int BK, int TA, int TB>
__global__ void __launch_bounds__(BM * BN / (T * T))
__attribute__((amdgpu_waves_per_eu(LpDmaCfg<EB, BM, BN, T, BK, TA, TB>::OCC, 8)))
gemm_lp_dma_kernel(GemmArgs args) {
  using Cfg = LpDmaCfg<EB, BM, BN, T, BK, TA, TB>;
  __shared__ __attribute__((aligned(16))) char lds[Cfg::LDS_BYTES];
  int tm, tn;
  int64_t bz;
  load_args(args);
  block_coords(blockIdx.x, args, tm, tn, bz);
  lp_dma_tile<EB, BM, BN, T, BK, TA, TB>(args, tm, tn, bz, lds);
}

// Operands whose rows all start on 16-byte boundaries take the DMA pipeline,
// any other the register-staged kernel.
template <int EB, int BM, int BN, int T, int BK, int TA, int TB>
hipError_t launch_gemm_lp(const GemmArgs& a, hipStream_t stream) {
  using Cfg = GemmLpCfg<EB, BM, BN, T, BK, TA, TB>;
  if (a.alignA == ROWS_16 && a.alignB == ROWS_16)
    return launch_flat<EB>(gemm_lp_dma_kernel<EB, BM, BN, T, BK, TA, TB>, a, BM, BN, Cfg::NT,
                           stream);
  return launch_flat<EB>(gemm_lp_kernel<EB, BM, BN, T, BK, TA, TB>, a, BM, BN, Cfg::NT, stream);
}

}  // namespace kt
