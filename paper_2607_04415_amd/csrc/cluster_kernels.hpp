// Kernels of the cluster placement: nearest centroids through the matrix
// units, a stable counting sort by cluster, and the centroid means.
#pragma once

#include <algorithm>

#include "wave.hpp"

namespace gorio {

// ---------------------------------------------------------------------------
// nearest centroid
// ---------------------------------------------------------------------------
// The score of centroid k for vector x is |c_k|^2 - 2 x . c_k with the dot
// product summed in d order, multiply and add rounded separately; the nearest
// centroid is the least score, ties to the smaller k.
__device__ __forceinline__ float centroid_score(float cc, float dot) {
  return __fsub_rn(cc, __fmul_rn(2.0f, dot));
}

// One thread per vector; every lane of a wave reads the same centroid element
// (a broadcast).  With the dimension known at compile time (DC > 0) the vector
// is held in registers and each centroid is read once per wave through scalar
// loads.  For calls with few vectors or centroids (query ordering).
template <typename T, int DC>
__global__ __launch_bounds__(256) void nearest_centroid(const T *v, uint64_t count, uint32_t D, const float *c,
                                                        const float *cc, uint32_t K, uint32_t *out) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const T *x = v + i * D;
  float best = 0.0f;
  uint32_t arg = 0;
  if constexpr (DC > 0) {
    float xr[DC];
#pragma unroll
    for (int d = 0; d < DC; ++d) xr[d] = (float)x[d];
    for (uint32_t k = 0; k < K; ++k) {
      const float *ck = c + (uint64_t)k * DC;
      float dot = 0.0f;
#pragma unroll
      for (int d = 0; d < DC; ++d) dot += xr[d] * ck[d];
      const float s = centroid_score(cc[k], dot);
      if (k == 0 || s < best) {
        best = s;
        arg = k;
      }
    }
  } else {
    for (uint32_t k = 0; k < K; ++k) {
      const float *ck = c + (uint64_t)k * D;
      float dot = 0.0f;
      for (uint32_t d = 0; d < D; ++d) dot += (float)x[d] * ck[d];
      const float s = centroid_score(cc[k], dot);
      if (k == 0 || s < best) {
        best = s;
        arg = k;
      }
    }
  }
  out[i] = arg;
}

// Centroids laid out for the matrix path: rows of DP floats (zeros past D),
// a whole number of 32-row tiles; scores of the padding rows are +inf.  Also
// the transposed rows (Kp floats per dimension), the squared norms in d order,
// a hash of each centroid's bits, and the largest norm's bits (a NaN's compare
// above every number's).
__global__ __launch_bounds__(64) void centroid_layouts(const float *c, uint32_t K, uint32_t D, uint32_t DP, uint32_t Kp,
                                                       float *rows, float *cols, float *cc, uint64_t *hash,
                                                       unsigned int *most) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= Kp) return;
  float s = 0.0f;
  uint64_t h = 0;
#pragma unroll 8
  for (uint32_t d = 0; d < DP; ++d) {
    const float x = k < K && d < D ? c[(uint64_t)k * D + d] : 0.0f;
    rows[(uint64_t)k * DP + d] = x;
    if (d < D) {
      cols[(uint64_t)d * Kp + k] = x;
      s = __fadd_rn(s, __fmul_rn(x, x));
      h = (h ^ __float_as_uint(x)) * 0x9E3779B97F4A7C15ull;
      h ^= h >> 29;
    }
  }
  hash[k] = h;
  cc[k] = k < K ? s : __uint_as_float(0x7F800000u);
  if (k < K) atomicMax(most, __float_as_uint(s) & 0x7FFFFFFFu);
}

// A centroid with the bits of an earlier one never wins (equal scores, larger
// index), but its ties would send every vector near it to the exact scores: its
// norm becomes +inf.  A wave per centroid looks for the first earlier one with
// its hash and compares the two; a hash in common with a different centroid
// leaves it as it is.  (1M x 128 uint8, all rows equal, 512 clusters, four
// iterations: 39.6 ms a call without, 12.7 with.)
__global__ __launch_bounds__(kWave) void drop_repeats(const float *c, uint32_t D, const uint64_t *hash, float *cc) {
  const uint32_t k = blockIdx.x, l = lane_id();
  const uint64_t h = hash[k];
  for (uint32_t j0 = 0; j0 < k; j0 += kWave) {
    const uint64_t m = ballot(j0 + l < k && hash[j0 + l] == h);
    if (m == 0) continue;
    const uint32_t j = j0 + (uint32_t)__builtin_ctzll(m);
    bool same = true;
    for (uint32_t d = l; d < D; d += kWave)
      same = same && __float_as_uint(c[(uint64_t)j * D + d]) == __float_as_uint(c[(uint64_t)k * D + d]);
    if (ballot(!same) == 0 && l == 0) cc[k] = __uint_as_float(0x7F800000u);
    return;
  }
}

// How far two computations of one score may lie apart on either side, twice:
// if the runner-up's matrix score is farther than this above the least one,
// the least one is also least in the stated order.  A dot product's rounding
// error is at most (D + 2) u sum |x_d c_d| <= (D + 2) u |x| |c| in any order of
// multiplies and adds (u = 2^-24); the matrix units get twice that, the norms'
// own error and the subtraction's the rest.  The last term covers products
// below the smallest normal number.
__device__ __forceinline__ float score_margin(uint32_t D, float xx, float cmax2) {
  const float u = 5.9604645e-8f;
  // (NaN, or squares near the top of the range: every vector is scored exactly)
  if (!(xx < 1e36f) || !(cmax2 < 1e36f)) return __uint_as_float(0x7F800000u);
  const float xn = sqrtf(xx) * 1.001f, cn = sqrtf(cmax2) * 1.001f;
  return 2.0f * u * (6.0f * (float)(D + 8) * xn * cn + 4.0f * cmax2) + 1e-30f * (1.0f + xn + cn);
}

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The three least scores of a vector so far and the first two's centroids.
struct Top3 {
  float s0, s1, s2;
  uint32_t k0, k1;
  __device__ __forceinline__ void add(float s, uint32_t k) {
    const bool b0 = s < s0, b1 = s < s1;
    s2 = __builtin_amdgcn_fmed3f(s1, s2, s);
    s1 = __builtin_amdgcn_fmed3f(s0, s1, s);
    k1 = b0 ? k0 : (b1 ? k : k1);
    k0 = b0 ? k : k0;
    s0 = fminf(s0, s);
  }
};

// Matrix path: a wave scores 32 NT vectors against 32 centroids at a time
// with v_mfma_f32_32x32x2f32 (vectors in the columns, held in registers;
// centroids in the rows, one tile at a time through LDS for the block's four
// waves) and keeps each vector's three least scores.  These sums are not in
// the stated order, so a vector is settled only when its runner-up lies
// farther off than score_margin; where only two centroids are that close the
// vector goes to `pairs`, else to `open`, and they are scored again exactly.
// The result is the stated one whatever the matrix units round.
// Bound by the matrix units: 2 n K D operations at 64 per cycle and SIMD.  1M
// x 128 against 512 centroids: 4.03 ms with the plain kernel (83% of the vector
// units' issue limit), 1.35 ms here (97 TFLOP/s; the selects of the three
// least take most of the rest) and 0.12 ms for the vectors scored again.
template <typename T, int DQ, int NT>
__global__ __launch_bounds__(256, 2) void nearest_matrix(const T *v, uint64_t count, uint32_t D, const float *rows,
                                                      const float *cc, uint32_t Kp, const unsigned int *most,
                                                      uint32_t *out, uint32_t *alt, uint32_t *pairs, uint32_t *open,
                                                      unsigned int *counts) {
  constexpr int DP = 8 * DQ;
  constexpr int kRow = DP + 4;  // floats per tile row in LDS: 16 rows' reads cover all banks
  constexpr int kPer = 32 * DP / 4 / 256;  // float4s a thread moves per tile
  static_assert(32 * DP / 4 % 256 == 0, "whole float4s per thread");
  __shared__ __align__(16) float tile[2][32 * kRow];
  __shared__ __align__(16) float tcc[2][32];
  const int l = lane_id(), w = threadIdx.x / kWave;
  const int col = l & 31, h = l >> 5;
  const uint64_t base = ((uint64_t)blockIdx.x * 4 + w) * (32 * NT);
  float x[NT][DQ][4];
  float margin[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const uint64_t i = base + n * 32 + col;
    const T *p = v + (i < count ? i : count - 1) * D;
    float xx = 0.0f;
    const bool whole = D % 4 == 0;  // rows start on, and end with, whole fours
#pragma unroll
    for (int q = 0; q < DQ; ++q) {
      const uint32_t d0 = 8 * q + 4 * h;
      float f[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (whole) {
        if (d0 < D) {
          if constexpr (sizeof(T) == 1) {
            const uint32_t b = *reinterpret_cast<const uint32_t *>(p + d0);
#pragma unroll
            for (int t = 0; t < 4; ++t) f[t] = (float)((b >> (8 * t)) & 0xFFu);
          } else {
            const float4 b = *reinterpret_cast<const float4 *>(p + d0);
            f[0] = b.x;
            f[1] = b.y;
            f[2] = b.z;
            f[3] = b.w;
          }
        }
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (d0 + t < D) f[t] = (float)p[d0 + t];
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        x[n][q][t] = f[t];
        xx += f[t] * f[t];
      }
    }
    xx += __shfl_xor(xx, 32);
    margin[n] = score_margin(D, xx, __uint_as_float(*most));
  }
  Top3 top[NT];
  const float inf = __uint_as_float(0x7F800000u);
#pragma unroll
  for (int n = 0; n < NT; ++n) top[n] = {inf, inf, inf, 0, 0};
  const uint32_t tiles = Kp / 32;
  const f32x4 *src = reinterpret_cast<const f32x4 *>(rows);
  f32x4 st[kPer];
  auto fetch = [&](uint32_t t) {
#pragma unroll
    for (int j = 0; j < kPer; ++j) st[j] = src[(uint64_t)t * (32 * DP / 4) + j * 256 + threadIdx.x];
  };
  auto store = [&](uint32_t t) {
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int e = j * 256 + threadIdx.x, r = e / (DP / 4), q = e % (DP / 4);
      *reinterpret_cast<f32x4 *>(&tile[t & 1][r * kRow + 4 * q]) = st[j];
    }
    if (threadIdx.x < 32) tcc[t & 1][threadIdx.x] = cc[t * 32 + threadIdx.x];
  };
  fetch(0);
  store(0);
  for (uint32_t t = 0; t < tiles; ++t) {
    __syncthreads();  // tile t is written; tile t - 1's readers are done
    if (t + 1 < tiles) fetch(t + 1);
    f32x16 acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[n][r] = 0.0f;
    const float *row = &tile[t & 1][col * kRow + 4 * h];
#pragma unroll
    for (int q = 0; q < DQ; ++q) {
      const float4 a = *reinterpret_cast<const float4 *>(row + 8 * q);
      const float av[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NT; ++n)
          acc[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], x[n][q][e], acc[n], 0, 0, 0);
    }
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const float4 c4 = *reinterpret_cast<const float4 *>(&tcc[t & 1][8 * r4 + 4 * h]);
      const float cv[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NT; ++n)
          top[n].add(centroid_score(cv[e], acc[n][4 * r4 + e]), t * 32 + 8 * r4 + 4 * h + e);
    }
    if (t + 1 < tiles) store(t + 1);
  }
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    // the other half of the wave holds the other rows of every tile
    Top3 o;
    o.s0 = __shfl_xor(top[n].s0, 32);
    o.s1 = __shfl_xor(top[n].s1, 32);
    o.s2 = __shfl_xor(top[n].s2, 32);
    o.k0 = (uint32_t)__shfl_xor((int)top[n].k0, 32);
    o.k1 = (uint32_t)__shfl_xor((int)top[n].k1, 32);
    top[n].add(o.s0, o.k0);
    top[n].add(o.s1, o.k1);
    top[n].s2 = fminf(top[n].s2, o.s2);
    const uint64_t i = base + n * 32 + col;
    const bool mine = h == 0 && i < count;
    // comparisons fail on NaN: such a vector is open
    const float limit = top[n].s0 + margin[n];
    const bool settled = top[n].s1 > limit, pair = !settled && top[n].s2 > limit;
    if (mine) {
      out[i] = top[n].k0;
      if (pair) alt[i] = top[n].k1;
    }
#pragma unroll
    for (int which = 0; which < 2; ++which) {
      const bool put = mine && (which == 0 ? pair : !settled && !pair);
      const uint64_t m = ballot(put);
      if (m == 0) continue;
      uint32_t at = 0;
      if (l == __builtin_ctzll(m)) at = atomicAdd(&counts[which], (unsigned int)__popcll(m));
      at = readlane(at, __builtin_ctzll(m)) + lanes_below(m);
      if (put) (which == 0 ? pairs : open)[at] = (uint32_t)i;
    }
  }
}

// The stated score of two centroids for each vector of the list.
template <typename T>
__global__ __launch_bounds__(256) void nearest_of_pair(const T *v, uint32_t D, const float *c, const float *cc,
                                                       const uint32_t *pairs, const unsigned int *count,
                                                       const uint32_t *alt, uint32_t *out) {
  const uint32_t n = *count;
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
    const uint32_t i = pairs[j];
    const uint32_t a = min(out[i], alt[i]), b = max(out[i], alt[i]);
    const T *x = v + (uint64_t)i * D;
    const float *ca = c + (uint64_t)a * D, *cb = c + (uint64_t)b * D;
    float da = 0.0f, db = 0.0f;
#pragma unroll 8
    for (uint32_t d = 0; d < D; ++d) {
      const float e = (float)x[d];
      da = __fadd_rn(da, __fmul_rn(e, ca[d]));
      db = __fadd_rn(db, __fmul_rn(e, cb[d]));
    }
    out[i] = centroid_score(cc[b], db) < centroid_score(cc[a], da) ? b : a;
  }
}

// The stated scores of all centroids for each vector of the list: a wave
// takes kOpenVecs vectors, its lanes 64 centroids at a time (the transposed
// rows make their loads whole lines).
constexpr int kOpenVecs = 8;
template <typename T>
__global__ __launch_bounds__(kWave) void nearest_of_all(const T *v, uint32_t D, const float *cols, const float *cc,
                                                        uint32_t K, uint32_t Kp, const uint32_t *open,
                                                        const unsigned int *count, uint32_t *out) {
  __shared__ float xs[256 * kOpenVecs];  // D <= 256
  const uint32_t n = *count, l = lane_id();
  for (uint32_t j0 = blockIdx.x * kOpenVecs; j0 < n; j0 += gridDim.x * kOpenVecs) {
    __syncthreads();
    for (uint32_t e = l; e < D * kOpenVecs; e += kWave) {
      const uint32_t d = e / kOpenVecs, j = min(j0 + e % kOpenVecs, n - 1);
      xs[e] = (float)v[(uint64_t)open[j] * D + d];
    }
    __syncthreads();
    // the scan's `k == 0 || s < best` from the left: lane l meets its
    // centroids in ascending order; a NaN score of centroid 0 stands
    float best[kOpenVecs];
    uint32_t arg[kOpenVecs];
    bool stuck[kOpenVecs];
#pragma unroll
    for (int j = 0; j < kOpenVecs; ++j) {
      best[j] = __uint_as_float(0x7F800000u);
      arg[j] = 0xFFFFFFFFu;
      stuck[j] = false;
    }
    for (uint32_t k0 = 0; k0 < K; k0 += kWave) {
      const uint32_t k = k0 + l, kc = min(k, Kp - 1);
      float dot[kOpenVecs];
#pragma unroll
      for (int j = 0; j < kOpenVecs; ++j) dot[j] = 0.0f;
#pragma unroll 4
      for (uint32_t d = 0; d < D; ++d) {
        const float cv = cols[(uint64_t)d * Kp + kc];
#pragma unroll
        for (int j = 0; j < kOpenVecs; ++j)
          dot[j] = __fadd_rn(dot[j], __fmul_rn(xs[d * kOpenVecs + j], cv));
      }
      if (k < K) {
#pragma unroll
        for (int j = 0; j < kOpenVecs; ++j) {
          const float s = centroid_score(cc[k], dot[j]);
          stuck[j] = stuck[j] || (k == 0 && !(s == s));
          if (s < best[j] || (arg[j] == 0xFFFFFFFFu && s == best[j])) {
            best[j] = s;
            arg[j] = k;
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kOpenVecs; ++j) {
      float b = best[j];
      uint32_t a = arg[j];
      for (int m = 1; m < kWave; m <<= 1) {
        const float ob = __shfl_xor(b, m);
        const uint32_t oa = (uint32_t)__shfl_xor((int)a, m);
        if (ob < b || (ob == b && oa < a)) {
          b = ob;
          a = oa;
        }
      }
      // no centroid below the first one: every score NaN, or the first NaN
      if (ballot(stuck[j]) != 0 || a == 0xFFFFFFFFu) a = 0;
      if (l == 0 && j0 + j < n) out[open[j0 + j]] = a;
    }
  }
}

// ---------------------------------------------------------------------------
// stable counting sort by cluster
// ---------------------------------------------------------------------------
// A wave takes `tile` consecutive nodes, 64 at a time: nodes of one cluster
// in the same 64 are ranked by their lanes, the first of them takes the
// cluster's count so far from the tile's row of `hist`.  Leaves each node's
// rank among its cluster's nodes of the tile, and the tile's counts.
__global__ __launch_bounds__(kWave) void tile_ranks(const uint32_t *key, uint32_t n, uint32_t K, uint32_t key_bits,
                                                    uint32_t tile, uint32_t *hist, uint32_t *rank) {
  const uint32_t l = lane_id();
  uint32_t *row = hist + (uint64_t)blockIdx.x * K;
  const uint32_t i0 = blockIdx.x * tile, i1 = min(n, i0 + tile);
  for (uint32_t b = i0; b < i1; b += kWave) {
    const uint32_t i = b + l;
    const bool in = i < i1;
    const uint32_t k = in ? key[i] : 0u;
    uint64_t same = ballot(in);
    for (uint32_t bit = 0; bit < key_bits; ++bit) {
      const uint64_t m = ballot((k >> bit) & 1u);
      same &= (k >> bit) & 1u ? m : ~m;
    }
    const uint32_t below = lanes_below(same);
    uint32_t first = 0;
    if (in && below == 0) first = atomicAdd(&row[k], (uint32_t)__popcll(same));
    const int leader = in ? __builtin_ctzll(same) : 0;
    first = (uint32_t)__shfl((int)first, leader);
    if (in) rank[i] = first + below;
  }
}

// Per cluster: the tiles' counts become the counts of the tiles before them;
// total[k] = all.
__global__ __launch_bounds__(64) void tile_prefix(uint32_t *hist, uint32_t tiles, uint32_t K, uint32_t *total) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  uint32_t s = 0;
  uint32_t t = 0;
  for (; t + 16 <= tiles; t += 16) {
    uint32_t c[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) c[j] = hist[(uint64_t)(t + j) * K + k];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      hist[(uint64_t)(t + j) * K + k] = s;
      s += c[j];
    }
  }
  for (; t < tiles; ++t) {
    const uint32_t c = hist[(uint64_t)t * K + k];
    hist[(uint64_t)t * K + k] = s;
    s += c;
  }
  total[k] = s;
}

// start[k] = nodes in the clusters before k; start[K] = n.  One block.
__global__ __launch_bounds__(1024) void cluster_starts(const uint32_t *total, uint32_t K, uint32_t *start) {
  __shared__ uint32_t part[1024];
  const uint32_t t = threadIdx.x, each = (K + 1023) / 1024, k0 = min(K, t * each), k1 = min(K, k0 + each);
  uint32_t s = 0;
  for (uint32_t k = k0; k < k1; ++k) s += total[k];
  part[t] = s;
  __syncthreads();
  for (uint32_t d = 1; d < 1024; d <<= 1) {
    const uint32_t o = t >= d ? part[t - d] : 0u;
    __syncthreads();
    part[t] += o;
    __syncthreads();
  }
  uint32_t a = part[t] - s;
  for (uint32_t k = k0; k < k1; ++k) {
    start[k] = a;
    a += total[k];
  }
  if (t == 1023) start[K] = part[1023];
}

// slot[i] = place of node i, order[slot] = i.
__global__ __launch_bounds__(256) void cluster_slots(const uint32_t *key, const uint32_t *rank, const uint32_t *hist,
                                                     const uint32_t *start, uint32_t n, uint32_t K, uint32_t tile,
                                                     uint32_t *slot, uint32_t *order) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t k = key[i];
  const uint32_t s = start[k] + hist[(uint64_t)(i / tile) * K + k] + rank[i];
  slot[i] = s;
  order[s] = i;
}

// ---------------------------------------------------------------------------
// centroid means
// ---------------------------------------------------------------------------
// uint8: the sums are whole numbers below 2^53, the same in any order.  A block
// takes `rows` places of the order, whatever clusters they belong to: a
// group of threads per row, V consecutive dimensions each, added up in LDS
// and then once per cluster in memory.  So a cluster that holds most nodes is
// shared among as many blocks as its rows need (1M x 128, all in one of 512
// clusters, four iterations: 92.9 ms a call with 16 blocks to a cluster, 39.6
// here; in one of one 25.2 and 6.4).
// About a thousand blocks, of 64 rows at least (a cluster's share costs four
// dependent loads; 20k nodes, 64 clusters, two iterations: 0.86 ms a call with
// 1,024 rows to a block, 0.75 so).
inline uint32_t sum_rows_u8(uint64_t n) { return (uint32_t)std::min<uint64_t>(1024, std::max<uint64_t>(64, n / 1024)); }
template <int V>
__global__ __launch_bounds__(256) void cluster_sums_u8(const uint8_t *v, uint32_t n, uint32_t D, uint32_t rows,
                                                       const uint32_t *order, const uint32_t *key,
                                                       const uint32_t *start, unsigned long long *sums) {
  __shared__ uint32_t part[1024];  // D <= 1024
  struct __align__(V) Unit { uint8_t e[V]; };
  const uint32_t units = D / V, groups = max(1u, blockDim.x / units);
  const uint32_t g = units < blockDim.x ? threadIdx.x / units : 0u, u0 = threadIdx.x - g * units;
  uint32_t p = blockIdx.x * rows;
  const uint32_t last = min(n, p + rows);
  while (p < last) {
    const uint32_t k = key[order[p]], p1 = min(last, start[k + 1]);
    for (uint32_t d = threadIdx.x; d < D; d += blockDim.x) part[d] = 0;
    __syncthreads();
    if (g < groups) {
      for (uint32_t u = u0; u < units; u += blockDim.x) {
        uint32_t s[V] = {};
#pragma unroll 8
        for (uint32_t i = p + g; i < p1; i += groups) {
          const Unit x = *reinterpret_cast<const Unit *>(v + (uint64_t)order[i] * D + u * V);
#pragma unroll
          for (int j = 0; j < V; ++j) s[j] += x.e[j];
        }
#pragma unroll
        for (int j = 0; j < V; ++j) atomicAdd(&part[u * V + j], s[j]);
      }
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < D; d += blockDim.x)
      if (part[d]) atomicAdd(&sums[(uint64_t)k * D + d], (unsigned long long)part[d]);
    __syncthreads();
    p = max(p + 1, p1);
  }
}

// float32: sums in float64 in a stated order: the nodes in kMeanRanges ranges,
// each range's members of a cluster in id order, then the ranges' sums in range
// order.  Block 16 k + t: the members of cluster k in range t, one thread per
// dimension; kFly rows are in flight while the kFly before them are added, and
// their ids a step earlier, so that a cluster that holds most nodes costs one
// memory trip per kFly rows (500k x 96, all in one of 256 clusters, four
// iterations: 34.3 ms a call with 8 rows loaded and then added, 20.5 here).
constexpr uint32_t kMeanRanges = 16;

__global__ __launch_bounds__(256) void cluster_sums_f32(const float *v, uint64_t n, uint32_t D, const uint32_t *order,
                                                        const uint32_t *start, double *sums) {
  const uint32_t t = blockIdx.x % kMeanRanges, k = blockIdx.x / kMeanRanges, K = gridDim.x / kMeanRanges;
  const uint32_t first = (uint32_t)(n * t / kMeanRanges), last = (uint32_t)(n * (t + 1) / kMeanRanges);
  auto lower = [&](uint32_t id) {  // first member of the cluster at or past id
    uint32_t a = start[k], b = start[k + 1];
    while (a < b) {
      const uint32_t m = a + (b - a) / 2;
      if (order[m] < id) a = m + 1;
      else b = m;
    }
    return first_lane_value(a);
  };
  const uint32_t p0 = lower(first), p1 = lower(last);
  constexpr int kFly = 32;
  for (uint32_t d = threadIdx.x; d < D; d += blockDim.x) {
    double s = 0.0;
    if (p0 < p1) {
      uint32_t id[kFly];
      float now[kFly], next[kFly];
      auto ids = [&](uint32_t p) {  // past the members: the last one again
#pragma unroll
        for (int f = 0; f < kFly; ++f) id[f] = order[min(p + f, p1 - 1)];
      };
      auto rows = [&](float (&x)[kFly]) {
#pragma unroll
        for (int f = 0; f < kFly; ++f) x[f] = v[(uint64_t)id[f] * D + d];
      };
      ids(p0);
      rows(now);
      ids(p0 + kFly);
      for (uint32_t p = p0; p < p1; p += kFly) {
        if (p + kFly < p1) rows(next);
        if (p + 2 * kFly < p1) ids(p + 2 * kFly);
        const uint32_t m = min((uint32_t)kFly, p1 - p);
        if (m == kFly) {
#pragma unroll
          for (int f = 0; f < kFly; ++f) s = __dadd_rn(s, (double)now[f]);
        } else {
#pragma unroll
          for (int f = 0; f < kFly; ++f)
            if ((uint32_t)f < m) s = __dadd_rn(s, (double)now[f]);
        }
#pragma unroll
        for (int f = 0; f < kFly; ++f) now[f] = next[f];
      }
    }
    sums[((uint64_t)t * K + k) * D + d] = s;
  }
}

// Each centroid becomes the mean of its members (an empty cluster keeps its
// centroid).
__global__ __launch_bounds__(256) void cluster_means_u8(const unsigned long long *sums, const uint32_t *start,
                                                        uint32_t K, uint32_t D, float *c) {
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (uint64_t)K * D) return;
  const uint32_t k = (uint32_t)(e / D);
  const uint32_t cnt = start[k + 1] - start[k];
  if (cnt != 0) c[e] = (float)__ddiv_rn((double)sums[e], (double)cnt);
}
__global__ __launch_bounds__(256) void cluster_means_f32(const double *sums, const uint32_t *start, uint32_t K,
                                                         uint32_t D, float *c) {
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (uint64_t)K * D) return;
  const uint32_t k = (uint32_t)(e / D);
  const uint32_t cnt = start[k + 1] - start[k];
  if (cnt == 0) return;
  double s = 0.0;
#pragma unroll
  for (uint32_t t = 0; t < kMeanRanges; ++t) s = __dadd_rn(s, sums[(uint64_t)t * K * D + e]);
  c[e] = (float)__ddiv_rn(s, (double)cnt);
}

__global__ void fill_words(uint32_t *w, uint64_t n, uint32_t value) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    w[i] = value;
}

}  // namespace gorio
