// Pruning of the configuration space on the GPU (sections 3.4, 4.1 and 4.2 of
// the paper): normalize the benchmark table, cluster its rows with k-means
// and turn each centroid into one deployed configuration.
//
// Everything is integer so that any correct implementation reaches the same
// bits: Q16 normalized values, exact int64 squared distances and sums,
// rounded-mean centroids floor((2*sum + n_j) / (2*n_j)), lowest index on every
// tie.  k-means++ initialisation draws from a SplitMix64 stream seeded with
// seed + restart.  One work-group runs one restart; restarts run in parallel.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "kt_internal.hpp"

namespace kt {

static constexpr int Q16 = 65535;
static constexpr int STD_LO = 58982;   // ceil(0.9 * 65535)

// ----------------------------------------------------------- normalization

// One work-group per row: t_best = smallest positive time of the row, then
// q = floor((2*65535*t_best + t) / (2*t)) and the chosen variant.
__global__ void __launch_bounds__(256)
normalize_kernel(const int64_t* __restrict__ T, int32_t n_cfg, int32_t norm,
                 const uint16_t* __restrict__ lut, uint16_t* __restrict__ out) {
  const int64_t row = blockIdx.x;
  const int64_t* t = T + row * n_cfg;
  __shared__ int64_t red[256];
  int64_t best = INT64_MAX;
  for (int c = threadIdx.x; c < n_cfg; c += blockDim.x) {
    const int64_t v = t[c];
    if (v > 0 && v < best) best = v;
  }
  red[threadIdx.x] = best;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s && red[threadIdx.x + s] < red[threadIdx.x]) red[threadIdx.x] = red[threadIdx.x + s];
    __syncthreads();
  }
  best = red[0];
  for (int c = threadIdx.x; c < n_cfg; c += blockDim.x) {
    const int64_t v = t[c];
    int64_t q = 0;
    if (v > 0 && best != INT64_MAX) q = (2 * (int64_t)Q16 * best + v) / (2 * v);
    if (norm == KT_NORM_RAWCUT) {
      if (10 * q < 9 * (int64_t)Q16) q = 0;
    } else if (norm == KT_NORM_STDCUT) {
      if (10 * q < 9 * (int64_t)Q16) q = 0;
      else {
        const int64_t num = (q - STD_LO) * Q16, den = Q16 - STD_LO;
        q = (2 * num + den) / (2 * den);
      }
    } else if (norm == KT_NORM_SIGMOID) {
      q = lut[q];
    }
    out[row * n_cfg + c] = (uint16_t)q;
  }
}

const std::vector<uint16_t>& sigmoid_table(Ctx* h) {
  if (h->sigmoid_lut.empty()) {
    h->sigmoid_lut.resize(Q16 + 1);
    for (int v = 0; v <= Q16; ++v) {
      const double f = (double)Q16 / (1.0 + exp(50.0 * (0.85 - (double)v / Q16)));
      h->sigmoid_lut[v] = (uint16_t)floor(f + 0.5);
    }
  }
  return h->sigmoid_lut;
}

// ------------------------------------------------------------------ k-means

static constexpr int KM_THREADS = 1024;
static constexpr int KM_MAX_ROWS = 4096;
static constexpr int KM_MAX_KD = 8192;      // k * d member sums in LDS

struct KmeansOut {      // per restart, in the workspace
  int64_t inertia;
  int32_t iterations;
  int32_t pad;
};

__device__ __forceinline__ uint64_t sm64_next(uint64_t& state) {
  uint64_t z = state + 0x9E3779B97F4A7C15ull;
  state = z;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Block-wide argmax of val[i] over i < n, lowest index on ties.
__device__ void block_argmax(const int64_t* val, int n, int64_t* s_val, int32_t* s_idx,
                             int64_t& out_val, int32_t& out_idx) {
  const int tid = threadIdx.x;
  int64_t bv = INT64_MIN;
  int32_t bi = INT32_MAX;
  for (int i = tid; i < n; i += KM_THREADS) {
    if (val[i] > bv) { bv = val[i]; bi = i; }   // ascending i: first max kept
  }
  s_val[tid] = bv;
  s_idx[tid] = bi;
  __syncthreads();
  for (int s = KM_THREADS / 2; s > 0; s >>= 1) {
    if (tid < s) {
      const int64_t ov = s_val[tid + s];
      const int32_t oi = s_idx[tid + s];
      if (ov > s_val[tid] || (ov == s_val[tid] && oi < s_idx[tid])) { s_val[tid] = ov; s_idx[tid] = oi; }
    }
    __syncthreads();
  }
  out_val = s_val[0];
  out_idx = s_idx[0];
  __syncthreads();
}

__device__ int64_t block_sum(int64_t v, int64_t* s_val) {
  const int tid = threadIdx.x;
  s_val[tid] = v;
  __syncthreads();
  for (int s = KM_THREADS / 2; s > 0; s >>= 1) {
    if (tid < s) s_val[tid] += s_val[tid + s];
    __syncthreads();
  }
  const int64_t r = s_val[0];
  __syncthreads();
  return r;
}

// The clustering works on the INT8 matrix cores.  A 16-bit value is
// x = 256 (a + 128) + (b + 128) with signed bytes a, b, and the offset cancels
// in x - c, so with x' = 256 a + b
//   |x - c|^2 = sum x'^2 - 2 sum x' c' + sum c'^2,
//   x' c' = 65536 a_x a_c + 256 (a_x b_c + b_x a_c) + b_x b_c:
// four byte products, each an exact 32-bit sum of a 16x16x64 INT8 MFMA (at
// most 8192 terms of 2^14).  The 16 columns of one MFMA are the two bytes of
// eight centroids, its rows sixteen rows of X, once for each byte of X.
struct KmLayout {          // LDS of one restart, in bytes
  int kt;                  // column tiles: eight centroids each
  int dp;                  // dimensions in whole 64-deep steps
  int o_planes, o_sums, o_xx, o_dist, o_cc, o_val, o_labels, o_counts, o_idx, total;
  __host__ __device__ KmLayout(int n, int d, int k) {
    kt = (k + 7) / 8;
    dp = (d + 63) / 64 * 64;
    int o = 0;
    auto take = [&](int bytes) { const int at = o; o += (bytes + 15) / 16 * 16; return at; };
    o_planes = take(2 * k * dp);        // centroid bytes [column][dp]
    o_sums = take(k * d * 4);           // member sums, at most 4096 * 65535
    o_xx = take(n * 8);                 // sum x'^2 per row
    o_dist = take(n * 8);
    o_cc = take(kt * 8 * 8);            // sum c'^2 per centroid
    o_val = take(KM_THREADS * 8);
    o_labels = take(n);
    o_counts = take(k * 4);
    o_idx = take(KM_THREADS * 4);
    total = o;
  }
};

typedef int i32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4h __attribute__((ext_vector_type(4), aligned(2)));

// One lane's bytes of 16 consecutive values of row i from column c0: the
// high bytes in hi, the low ones in lo, both signed; zero beyond d.
__device__ __forceinline__ void km_load(const uint16_t* __restrict__ X, int d, int i, int c0,
                                        i32x4v& hi, i32x4v& lo) {
  const uint16_t* p = X + (int64_t)i * d + c0;
  uint32_t w[8];
  uint32_t keep[4];
  if (c0 + 16 <= d) {
    const u32x4h u = *reinterpret_cast<const u32x4h*>(p);
    const u32x4h v = *reinterpret_cast<const u32x4h*>(p + 8);
#pragma unroll
    for (int q = 0; q < 4; ++q) { w[q] = u[q]; w[4 + q] = v[q]; keep[q] = 0xffffffffu; }
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t e0 = c0 + 2 * q < d ? p[2 * q] : 0u, e1 = c0 + 2 * q + 1 < d ? p[2 * q + 1] : 0u;
      w[q] = e0 | (e1 << 16);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int left = d - c0 - 4 * q;
      keep[q] = left >= 4 ? 0xffffffffu : left <= 0 ? 0u : (1u << (8 * left)) - 1u;
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    hi[q] = (int)((__builtin_amdgcn_perm(w[2 * q + 1], w[2 * q], 0x07050301u) ^ 0x80808080u) & keep[q]);
    lo[q] = (int)((__builtin_amdgcn_perm(w[2 * q + 1], w[2 * q], 0x06040200u) ^ 0x80808080u) & keep[q]);
  }
}

// Dot products of 16 rows (tile t) with the eight centroids of column tile ct:
// in lane l, x'_row . c'_j for rows 4 (l / 16) + r, r = 0..3, and centroid
// j = 8 ct + (l % 16) / 2 (both lanes of a pair hold it).
__device__ __forceinline__ void km_dots(const uint16_t* __restrict__ X, int n, int d, int t, int ct,
                                        const char* planes, int dp, int k, int lane, int64_t dot[4]) {
  const int row = min(t * 16 + (lane & 15), n - 1), kg = (lane >> 4) * 16;
  i32x4v ah = {0, 0, 0, 0}, al = {0, 0, 0, 0};
  const char* bp = planes + min(ct * 16 + (lane & 15), 2 * k - 1) * dp + kg;   // spare columns: any
  for (int s = 0; s < dp; s += 64) {
    i32x4v hi, lo;
    km_load(X, d, row, s + kg, hi, lo);
    const i32x4v b = *reinterpret_cast<const i32x4v*>(bp + s);
    ah = __builtin_amdgcn_mfma_i32_16x16x64_i8(hi, b, ah, 0, 0, 0);
    al = __builtin_amdgcn_mfma_i32_16x16x64_i8(lo, b, al, 0, 0, 0);
  }
  const int sh = (lane & 1) ? 0 : 8;   // even columns hold the centroids' high bytes
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t v = ((int64_t)ah[r] * 256 + al[r]) << sh;
    dot[r] = v + __shfl_xor(v, 1);
  }
}

// Write centroid j (one value per dimension) as bytes and its sum c'^2, by
// one wave; value(f) gives dimension f.
template <typename F>
__device__ __forceinline__ void km_set_centroid(char* planes, int64_t* cc, int dp, int d, int j,
                                                int lane, F value) {
  int64_t q = 0;
  for (int f = lane; f < d; f += 64) {
    const uint32_t v = value(f);
    planes[(2 * j) * dp + f] = (char)((v >> 8) ^ 0x80u);
    planes[(2 * j + 1) * dp + f] = (char)((v & 0xffu) ^ 0x80u);
    const int64_t c = (int64_t)v - 32896;
    q += c * c;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o);
  if (lane == 0) cc[j] = q;
}

// One restart per work-group.  Outputs in global memory: centroids
// [restart][k][d], labels [restart][n], KmeansOut [restart].
//
// An iteration reads X ceil(k / 8) times from L2, once for each column tile (960 x
// 188, k = 8: 361 KB, 2.4 us at one CU's 64 B a clock and 2.4 GHz); the products are
// 360 MFMAs.  Rows that
// change their cluster move between the member sums as they are found, so the
// update costs the changed rows only (the sums are exact integers).  With 64-bit
// vector arithmetic and a serial pass over the rows per dimension the same ten
// restarts of 960 x 188, k = 8, took 33 ms, this way 1.5.
__global__ void __launch_bounds__(KM_THREADS)
kmeans_kernel(const uint16_t* __restrict__ X, int n, int d, int k, uint64_t seed, int max_iter,
              int64_t* __restrict__ g_cent, int32_t* __restrict__ g_labels,
              KmeansOut* __restrict__ g_out) {
  extern __shared__ __attribute__((aligned(16))) char km_lds[];
  const KmLayout L(n, d, k);
  char* planes = km_lds + L.o_planes;
  uint32_t* sums = (uint32_t*)(km_lds + L.o_sums);
  int64_t* xx = (int64_t*)(km_lds + L.o_xx);
  int64_t* dist = (int64_t*)(km_lds + L.o_dist);
  int64_t* cc = (int64_t*)(km_lds + L.o_cc);
  int64_t* s_val = (int64_t*)(km_lds + L.o_val);
  uint8_t* labels = (uint8_t*)(km_lds + L.o_labels);
  int32_t* counts = (int32_t*)(km_lds + L.o_counts);
  int32_t* s_idx = (int32_t*)(km_lds + L.o_idx);
  __shared__ int32_t s_flag;
  __shared__ int32_t s_pick;
  __shared__ int64_t s_target;
  __shared__ int32_t s_centres[64];
  constexpr uint8_t NO_LABEL = 255;   // k <= 64
  constexpr int WAVES = KM_THREADS / 64;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = blockIdx.x;
  const int tiles = (n + 15) / 16;
  uint64_t state = seed + (uint64_t)r;   // thread 0 owns the stream

  for (int e = tid; e < 2 * k * L.dp / 4; e += KM_THREADS) ((uint32_t*)planes)[e] = 0u;
  for (int e = tid; e < k * d; e += KM_THREADS) sums[e] = 0u;
  for (int j = tid; j < k; j += KM_THREADS) counts[j] = 0;
  for (int i = tid; i < n; i += KM_THREADS) { labels[i] = NO_LABEL; dist[i] = INT64_MAX; }
  for (int i = wave; i < n; i += WAVES) {
    int64_t q = 0;
    for (int f = lane; f < d; f += 64) {
      const int64_t v = (int64_t)X[(int64_t)i * d + f] - 32896;
      q += v * v;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o);
    if (lane == 0) xx[i] = q;
  }

  // ---- k-means++ initialisation
  if (tid == 0) {
    const uint64_t draw = sm64_next(state);
    s_pick = (int)(draw % (uint64_t)n);
    s_centres[0] = s_pick;
  }
  __syncthreads();
  for (int c = 0; c < k; ++c) {
    if (c > 0) {
      // each thread owns a contiguous chunk of rows; exclusive prefix sums of
      // the chunks place the draw
      const int chunk = (n + KM_THREADS - 1) / KM_THREADS;
      const int lo = min(n, tid * chunk), hi = min(n, lo + chunk);
      int64_t part = 0;
      for (int i = lo; i < hi; ++i) part += dist[i];
      int64_t run = part;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int64_t up = __shfl_up(run, o);
        if (lane >= o) run += up;
      }
      if (lane == 63) s_val[wave] = run;
      __syncthreads();
      int64_t before = 0, S = 0;
      for (int w = 0; w < WAVES; ++w) {
        if (w < wave) before += s_val[w];
        S += s_val[w];
      }
      if (tid == 0) {
        const uint64_t draw = sm64_next(state);
        s_target = S == 0 ? -1 : (int64_t)(draw % (uint64_t)S);
        s_pick = 0;
        if (S == 0) {   // every row coincides with a centre: the first unused row
          int pick = -1;
          for (int i = 0; i < n && pick < 0; ++i) {
            bool used = false;
            for (int j = 0; j < c; ++j) used = used || (s_centres[j] == i);
            if (!used) pick = i;
          }
          s_pick = pick < 0 ? 0 : pick;
        }
      }
      __syncthreads();
      const int64_t rr = s_target;
      const int64_t start = before + run - part;
      if (rr >= start && rr < start + part) {   // one thread: the chunks do not overlap
        int64_t acc = start;
        for (int i = lo; i < hi; ++i) {
          acc += dist[i];
          if (acc > rr) { s_pick = i; break; }
        }
      }
      __syncthreads();
      if (tid == 0) s_centres[c] = s_pick;
    }
    const int64_t pick = s_pick;
    if (wave == 0)
      km_set_centroid(planes, cc, L.dp, d, c, lane, [&](int f) { return (uint32_t)X[pick * d + f]; });
    __syncthreads();
    const int64_t ccj = cc[c];
    for (int t = wave; t < tiles; t += WAVES) {
      int64_t dot[4];
      km_dots(X, n, d, t, c / 8, planes, L.dp, k, lane, dot);
      if ((lane & 15) == 2 * (c % 8)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = t * 16 + (lane >> 4) * 4 + q;
          if (i < n) {
            const int64_t v = xx[i] + ccj - 2 * dot[q];
            if (v < dist[i]) dist[i] = v;
          }
        }
      }
    }
    __syncthreads();
  }

  // ---- Lloyd iterations
  int it = 0;
  for (;;) {
    // assignment: nearest centroid, lowest index on ties
    if (tid == 0) s_flag = 0;
    __syncthreads();
    bool changed = false;
    for (int t = wave; t < tiles; t += WAVES) {
      int64_t best[4];
      int bj[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { best[q] = INT64_MAX; bj[q] = 0; }
      for (int ct = 0; ct < L.kt; ++ct) {
        int64_t dot[4];
        km_dots(X, n, d, t, ct, planes, L.dp, k, lane, dot);
        const int j = ct * 8 + (lane & 15) / 2;
        const int64_t ccj = j < k ? cc[j] : 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t v = ccj - 2 * dot[q];
          if (j < k && v < best[q]) { best[q] = v; bj[q] = j; }
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int o = 2; o < 16; o <<= 1) {
          const int64_t ov = __shfl_xor(best[q], o);
          const int oj = __shfl_xor(bj[q], o);
          if (ov < best[q] || (ov == best[q] && oj < bj[q])) { best[q] = ov; bj[q] = oj; }
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = t * 16 + (lane >> 4) * 4 + q;
        const bool in = i < n;
        const int old = in ? labels[i] : 0;
        const bool moved = in && old != bj[q];
        if (in && (lane & 15) == 0) {
          dist[i] = best[q] + xx[i];
          if (moved) {
            labels[i] = (uint8_t)bj[q];
            atomicAdd(&counts[bj[q]], 1);
            if (old != NO_LABEL) atomicSub(&counts[old], 1);
          }
        }
        changed = changed || moved;
        // the rows that moved, one of each 16-lane group, by the whole wave
        uint64_t todo = __ballot(moved && (lane & 15) == 0);
        while (todo) {
          const int src = __ffsll((unsigned long long)todo) - 1;
          todo &= todo - 1;
          const int row = t * 16 + (src >> 4) * 4 + q;
          const int to = __shfl(bj[q], src), from = __shfl(old, src);
          for (int f = lane; f < d; f += 64) {
            const uint32_t v = X[(int64_t)row * d + f];
            atomicAdd(&sums[to * d + f], v);
            if (from != NO_LABEL) atomicSub(&sums[from * d + f], v);
          }
        }
      }
    }
    if (changed) atomicOr(&s_flag, 1);
    __syncthreads();
    if (s_flag == 0 && it > 0) break;
    if (it >= max_iter) break;   // labels/dist already reflect the final centroids
    // update: rounded means
    for (int j = wave; j < k; j += WAVES) {
      const uint64_t nj = counts[j];
      if (nj > 0)
        km_set_centroid(planes, cc, L.dp, d, j, lane, [&](int f) {
          return (uint32_t)((2 * (uint64_t)sums[j * d + f] + nj) / (2 * nj));
        });
    }
    __syncthreads();
    // empty clusters take the farthest row (lowest index on ties); its distance is zeroed
    for (int j = 0; j < k; ++j) {
      if (counts[j] != 0) continue;
      int64_t fv;
      int32_t fi;
      block_argmax(dist, n, s_val, s_idx, fv, fi);
      if (wave == 0)
        km_set_centroid(planes, cc, L.dp, d, j, lane,
                        [&](int f) { return (uint32_t)X[(int64_t)fi * d + f]; });
      if (tid == 0) dist[fi] = 0;
      __syncthreads();
    }
    ++it;
  }
  int64_t part = 0;
  for (int i = tid; i < n; i += KM_THREADS) part += dist[i];
  const int64_t inertia = block_sum(part, s_val);
  for (int e = tid; e < k * d; e += KM_THREADS) {
    const int j = e / d, f = e - j * d;
    const uint32_t hi = (uint8_t)planes[(2 * j) * L.dp + f] ^ 0x80u;
    const uint32_t lo = (uint8_t)planes[(2 * j + 1) * L.dp + f] ^ 0x80u;
    g_cent[(int64_t)r * k * d + e] = hi * 256 + lo;
  }
  for (int i = tid; i < n; i += KM_THREADS) g_labels[(int64_t)r * n + i] = labels[i];
  if (tid == 0) {
    g_out[r].inertia = inertia;
    g_out[r].iterations = it;
  }
}

// Pick the winning restart (lowest inertia, lowest restart on ties) and map
// its centroids to k distinct configurations: centroid j takes its largest
// coordinate (lowest configuration on ties) among those not yet chosen.
__global__ void __launch_bounds__(64)
choose_kernel(const int64_t* __restrict__ g_cent, const KmeansOut* __restrict__ g_out, int n_init,
              int k, int d, int32_t* __restrict__ chosen, int32_t* __restrict__ best_restart) {
  __shared__ int32_t s_chosen[64];
  const int lane = threadIdx.x;
  // lexicographic minimum / maximum over the wave, lowest index on ties
  auto best_of = [&](int64_t v, int i) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const int64_t ov = __shfl_xor(v, o);
      const int oi = __shfl_xor(i, o);
      if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
    }
    return i;
  };
  int64_t bv = INT64_MIN;
  int bi = INT32_MAX;
  for (int r = lane; r < n_init; r += 64) {
    const int64_t v = -g_out[r].inertia;
    if (v > bv) { bv = v; bi = r; }
  }
  const int br = best_of(bv, bi);
  if (lane == 0) *best_restart = br;
  const int64_t* C = g_cent + (int64_t)br * k * d;
  for (int j = 0; j < k; ++j) {
    bv = -1;   // below every coordinate
    bi = INT32_MAX;
    for (int f = lane; f < d; f += 64) {
      bool used = false;
      for (int q = 0; q < j; ++q) used = used || (s_chosen[q] == f);
      const int64_t v = C[(int64_t)j * d + f];
      if (!used && v > bv) { bv = v; bi = f; }
    }
    const int best = best_of(bv, bi);
    if (lane == 0) {
      s_chosen[j] = best == INT32_MAX ? -1 : best;
      chosen[j] = s_chosen[j];
    }
    __syncthreads();
  }
}

static size_t a256(size_t v) { return (v + 255) & ~(size_t)255; }

struct PrunePlan {
  size_t off_T, off_X, off_cent, off_lab, off_out, off_chosen, total;
};

static PrunePlan prune_plan(int32_t n, int32_t d, int32_t k, int32_t n_init) {
  PrunePlan p;
  p.off_T = 0;
  p.off_X = a256(p.off_T + (size_t)n * d * 8);
  p.off_cent = a256(p.off_X + (size_t)n * d * 2);
  p.off_lab = a256(p.off_cent + (size_t)n_init * k * d * 8);
  p.off_out = a256(p.off_lab + (size_t)n_init * n * 4);
  p.off_chosen = a256(p.off_out + (size_t)n_init * sizeof(KmeansOut));
  p.total = a256(p.off_chosen + (size_t)(k + 1) * 4);
  return p;
}

static size_t kmeans_lds_bytes(int n, int d, int k) { return (size_t)KmLayout(n, d, k).total; }

static kt_status check_table(Ctx* h, int32_t n, int32_t d) {
  if (n < 1 || d < 1) return fail(h, KT_EINVAL, "empty time table");
  return KT_OK;
}

// Upload a host table and normalize it into the workspace (shared by prune and Top-N).
static kt_status ensure_lut(Ctx* h, hipStream_t st);

static kt_status upload_normalize(Ctx* h, const int64_t* time_ns, int32_t n, int32_t d, kt_norm norm,
                                  char* ws, const PrunePlan& p, hipStream_t st) {
  kt_status s = ensure_lut(h, st);
  if (s != KT_OK) return s;
  hipError_t e = hipMemcpyAsync(ws + p.off_T, time_ns, (size_t)n * d * 8, hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return hip_fail(h, e, "upload time table");
  hipLaunchKernelGGL(normalize_kernel, dim3(n), dim3(256), 0, st, (const int64_t*)(ws + p.off_T), d,
                     (int32_t)norm, (const uint16_t*)h->d_lut, (uint16_t*)(ws + p.off_X));
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "normalize launch");
  return KT_OK;
}

// Device copy of the sigmoid table, owned by the handle (128 KiB, made once).
static kt_status ensure_lut(Ctx* h, hipStream_t st) {
  if (h->d_lut) return KT_OK;
  const std::vector<uint16_t>& lut = sigmoid_table(h);
  hipError_t e = hipMalloc(&h->d_lut, lut.size() * 2);
  if (e != hipSuccess) { h->d_lut = nullptr; return hip_fail(h, e, "hipMalloc sigmoid table"); }
  e = hipMemcpyAsync(h->d_lut, lut.data(), lut.size() * 2, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(h, e, "upload sigmoid table");
  return KT_OK;
}

kt_status normalize_table_host(Ctx* h, const int64_t* time_ns, int32_t n, int32_t d, kt_norm norm,
                               void* workspace, size_t ws_bytes, hipStream_t st, uint16_t* out) {
  if (!need_device(h)) return KT_EINVAL;
  kt_status s = check_table(h, n, d);
  if (s != KT_OK) return s;
  if ((int)norm < 0 || (int)norm > 3) return fail(h, KT_EINVAL, "bad normalization");
  const PrunePlan p = prune_plan(n, d, 1, 1);
  if (!workspace || ws_bytes < p.total) return fail(h, KT_EWORKSPACE, "normalization workspace too small");
  s = upload_normalize(h, time_ns, n, d, norm, (char*)workspace, p, st);
  if (s != KT_OK) return s;
  hipError_t e = hipMemcpyAsync(out, (char*)workspace + p.off_X, (size_t)n * d * 2,
                                hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(h, e, "read normalized table");
  return KT_OK;
}

}  // namespace kt

using namespace kt;

extern "C" {

kt_status kt_normalize(kt_handle hh, const int64_t* d_time, int32_t n_rows, int32_t n_configs,
                       kt_norm norm, uint16_t* d_out, void* stream) {
  Ctx* h = reinterpret_cast<Ctx*>(hh);
  if (!h) return fail(nullptr, KT_EINVAL, "NULL handle");
  if (!need_device(h)) return KT_EINVAL;
  if (n_rows < 0 || n_configs < 0) return fail(h, KT_EINVAL, "negative size");
  if ((int)norm < 0 || (int)norm > 3) return fail(h, KT_EINVAL, "bad normalization");
  if (n_rows == 0 || n_configs == 0) return KT_OK;
  if (!d_time || !d_out) return fail(h, KT_EINVAL, "NULL table");
  hipStream_t st = (hipStream_t)stream;
  kt_status s = ensure_lut(h, st);
  if (s != KT_OK) return s;
  hipLaunchKernelGGL(normalize_kernel, dim3(n_rows), dim3(256), 0, st, d_time, n_configs, (int32_t)norm,
                     (const uint16_t*)h->d_lut, d_out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "normalize launch");
  return KT_OK;
}

kt_status kt_prune_workspace_bytes(int32_t n_rows, int32_t n_configs, int32_t k, int32_t n_init,
                                   size_t* bytes) {
  if (!bytes || n_rows < 1 || n_configs < 1 || k < 1 || n_init < 1) return KT_EINVAL;
  *bytes = prune_plan(n_rows, n_configs, k, n_init).total;
  return KT_OK;
}

kt_status kt_prune(kt_handle hh, const int64_t* time_ns, int32_t n, int32_t d, int32_t k,
                   kt_norm norm, uint64_t seed, int32_t n_init, int32_t max_iter, void* workspace,
                   size_t ws_bytes, void* stream, int32_t* chosen, int64_t* inertia_out,
                   int32_t* labels, int64_t* centroids) {
  Ctx* h = reinterpret_cast<Ctx*>(hh);
  if (!h) return fail(nullptr, KT_EINVAL, "NULL handle");
  if (!need_device(h)) return KT_EINVAL;
  kt_status s = check_table(h, n, d);
  if (s != KT_OK) return s;
  if (!time_ns || !chosen || !inertia_out) return fail(h, KT_EINVAL, "NULL argument");
  if ((int)norm < 0 || (int)norm > 3) return fail(h, KT_EINVAL, "bad normalization");
  if (k < 1 || k > n || k > d || k > 64) return fail(h, KT_EINVAL, "need 1 <= k <= min(n_rows, n_configs, 64)");
  if (n_init < 1 || max_iter < 0) return fail(h, KT_EINVAL, "need n_init >= 1 and max_iter >= 0");
  if (n > KM_MAX_ROWS || (int64_t)k * d > KM_MAX_KD)
    return fail(h, KT_EUNSUPPORTED, "k-means limits: n_rows <= 4096 and k * n_configs <= 8192");
  const PrunePlan p = prune_plan(n, d, k, n_init);
  if (!workspace || ws_bytes < p.total) return fail(h, KT_EWORKSPACE, "prune workspace too small");
  char* ws = (char*)workspace;
  hipStream_t st = (hipStream_t)stream;
  s = upload_normalize(h, time_ns, n, d, norm, ws, p, st);
  if (s != KT_OK) return s;
  const size_t lds = kmeans_lds_bytes(n, d, k);
  hipError_t e = hipFuncSetAttribute((const void*)kmeans_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return hip_fail(h, e, "kmeans LDS attribute");
  hipLaunchKernelGGL(kmeans_kernel, dim3(n_init), dim3(KM_THREADS), lds, st,
                     (const uint16_t*)(ws + p.off_X), n, d, k, seed, max_iter,
                     (int64_t*)(ws + p.off_cent), (int32_t*)(ws + p.off_lab),
                     (KmeansOut*)(ws + p.off_out));
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "kmeans launch");
  int32_t* d_chosen = (int32_t*)(ws + p.off_chosen);
  hipLaunchKernelGGL(choose_kernel, dim3(1), dim3(64), 0, st, (const int64_t*)(ws + p.off_cent),
                     (const KmeansOut*)(ws + p.off_out), n_init, k, d, d_chosen, d_chosen + k);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "choose launch");
  std::vector<int32_t> hc(k + 1);
  e = hipMemcpyAsync(hc.data(), d_chosen, (size_t)(k + 1) * 4, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(h, e, "read chosen");
  const int br = hc[k];
  KmeansOut o;
  e = hipMemcpy(&o, ws + p.off_out + br * sizeof(KmeansOut), sizeof o, hipMemcpyDeviceToHost);
  if (e == hipSuccess && labels)
    e = hipMemcpy(labels, ws + p.off_lab + (size_t)br * n * 4, (size_t)n * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess && centroids)
    e = hipMemcpy(centroids, ws + p.off_cent + (size_t)br * k * d * 8, (size_t)k * d * 8,
                  hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_fail(h, e, "read k-means result");
  memcpy(chosen, hc.data(), (size_t)k * 4);
  *inertia_out = o.inertia;
  return KT_OK;
}

kt_status kt_kmeans_u16(kt_handle hh, const uint16_t* X, int32_t n, int32_t d, int32_t k,
                        uint64_t seed, int32_t n_init, int32_t max_iter, void* workspace,
                        size_t ws_bytes, void* stream, int32_t* labels, int64_t* centroids,
                        int64_t* inertia_out) {
  Ctx* h = reinterpret_cast<Ctx*>(hh);
  if (!h) return fail(nullptr, KT_EINVAL, "NULL handle");
  if (!need_device(h)) return KT_EINVAL;
  if (n < 1 || d < 1) return fail(h, KT_EINVAL, "need n >= 1 and d >= 1");
  if (!X || !labels || !inertia_out) return fail(h, KT_EINVAL, "NULL argument");
  if (k < 1 || k > n || k > 64) return fail(h, KT_EINVAL, "need 1 <= k <= min(n, 64)");
  if (n_init < 1 || max_iter < 0) return fail(h, KT_EINVAL, "need n_init >= 1 and max_iter >= 0");
  if (n > KM_MAX_ROWS || (int64_t)k * d > KM_MAX_KD)
    return fail(h, KT_EUNSUPPORTED, "k-means limits: n <= 4096 and k * d <= 8192");
  const PrunePlan p = prune_plan(n, d, k, n_init);
  if (!workspace || ws_bytes < p.total) return fail(h, KT_EWORKSPACE, "k-means workspace too small");
  char* ws = (char*)workspace;
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = hipMemcpyAsync(ws + p.off_X, X, (size_t)n * d * 2, hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return hip_fail(h, e, "upload vectors");
  const size_t lds = kmeans_lds_bytes(n, d, k);
  e = hipFuncSetAttribute((const void*)kmeans_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)lds);
  if (e != hipSuccess) return hip_fail(h, e, "kmeans LDS attribute");
  hipLaunchKernelGGL(kmeans_kernel, dim3(n_init), dim3(KM_THREADS), lds, st,
                     (const uint16_t*)(ws + p.off_X), n, d, k, seed, max_iter,
                     (int64_t*)(ws + p.off_cent), (int32_t*)(ws + p.off_lab),
                     (KmeansOut*)(ws + p.off_out));
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "kmeans launch");
  // the restart with the lowest inertia (its per-coordinate picks are unused)
  int32_t* d_chosen = (int32_t*)(ws + p.off_chosen);
  hipLaunchKernelGGL(choose_kernel, dim3(1), dim3(64), 0, st, (const int64_t*)(ws + p.off_cent),
                     (const KmeansOut*)(ws + p.off_out), n_init, k, d, d_chosen, d_chosen + k);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(h, e, "choose launch");
  int32_t br = 0;
  e = hipMemcpyAsync(&br, d_chosen + k, 4, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(h, e, "read best restart");
  KmeansOut o;
  e = hipMemcpy(&o, ws + p.off_out + br * sizeof(KmeansOut), sizeof o, hipMemcpyDeviceToHost);
  if (e == hipSuccess)
    e = hipMemcpy(labels, ws + p.off_lab + (size_t)br * n * 4, (size_t)n * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess && centroids)
    e = hipMemcpy(centroids, ws + p.off_cent + (size_t)br * k * d * 8, (size_t)k * d * 8,
                  hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_fail(h, e, "read k-means result");
  *inertia_out = o.inertia;
  return KT_OK;
}

kt_status kt_prune_topn(kt_handle hh, const int64_t* time_ns, int32_t n, int32_t d, int32_t k,
                        void* workspace, size_t ws_bytes, void* stream, int32_t* chosen) {
  Ctx* h = reinterpret_cast<Ctx*>(hh);
  if (!h) return fail(nullptr, KT_EINVAL, "NULL handle");
  if (!need_device(h)) return KT_EINVAL;
  kt_status s = check_table(h, n, d);
  if (s != KT_OK) return s;
  if (!time_ns || !chosen || k < 1 || k > d) return fail(h, KT_EINVAL, "bad arguments");
  const PrunePlan p = prune_plan(n, d, 1, 1);
  if (!workspace || ws_bytes < p.total) return fail(h, KT_EWORKSPACE, "Top-N workspace too small");
  hipStream_t st = (hipStream_t)stream;
  s = upload_normalize(h, time_ns, n, d, KT_NORM_RELATIVE, (char*)workspace, p, st);
  if (s != KT_OK) return s;
  std::vector<uint16_t> X((size_t)n * d);
  hipError_t e = hipMemcpyAsync(X.data(), (char*)workspace + p.off_X, X.size() * 2,
                                hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(h, e, "read normalized table");
  std::vector<int64_t> count(d, 0);
  for (int32_t i = 0; i < n; ++i) {
    const uint16_t* x = &X[(size_t)i * d];
    int best = 0;
    for (int f = 1; f < d; ++f) if (x[f] > x[best]) best = f;
    count[best]++;
  }
  std::vector<int32_t> order(d);
  for (int f = 0; f < d; ++f) order[f] = f;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return count[a] > count[b]; });
  for (int j = 0; j < k; ++j) chosen[j] = order[j];
  return KT_OK;
}

}  // extern "C"
