// Index construction on the GPU: page packing, layout checks and the medoid
// entry rule.
#pragma once

#include "common.hpp"
#include "ordered_sum.hpp"

namespace gorio {

// Byte fill (the packed page array starts zeroed: page tails are zero).
__global__ void fill_u32(uint32_t *dst, uint64_t words, uint32_t value) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
       i += (uint64_t)gridDim.x * blockDim.x)
    dst[i] = value;
}

// node_to_slot must be a permutation of [0, n): count out-of-range or repeated slots.
__global__ void check_permutation(const uint32_t *node_to_slot, uint32_t n, uint32_t *seen_bits,
                                  unsigned int *bad) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    uint32_t s = node_to_slot[i];
    if (s >= n) { atomicAdd(bad, 1u); continue; }
    uint32_t bit = 1u << (s & 31);
    uint32_t old = atomicOr(&seen_bits[s >> 5], bit);
    if (old & bit) atomicAdd(bad, 1u);
  }
}

// One wave per node: copy the vector, compact the real edges (UINT32_MAX =
// no edge) in order, pad with UINT32_MAX, store the degree.  Ids >= n that
// are not UINT32_MAX are counted in *bad.
__global__ __launch_bounds__(256) void pack_records(const uint8_t *vectors, uint32_t vec_bytes,
                                                    const uint32_t *graph, uint32_t R, uint32_t n,
                                                    PageGeom geom, uint8_t *pages, unsigned int *bad) {
  const int l = lane_id();
  const uint32_t waves = gridDim.x * (blockDim.x / kWave);
  for (uint32_t v = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; v < n; v += waves) {
    const uint32_t s = slot_of(geom, v);
    const uint32_t *src = reinterpret_cast<const uint32_t *>(vectors + (uint64_t)v * vec_bytes);
    uint32_t *dst = reinterpret_cast<uint32_t *>(pages + vec_offset(geom, s));
    for (uint32_t w = l; w < vec_bytes / 4; w += kWave) dst[w] = src[w];
    uint8_t *adj = pages + adj_offset(geom, s);
    uint32_t *ids = reinterpret_cast<uint32_t *>(adj + 4);
    uint32_t deg = 0;
    for (uint32_t j0 = 0; j0 < R; j0 += kWave) {
      uint32_t j = j0 + l;
      uint32_t id = j < R ? graph[(uint64_t)v * R + j] : kNoEdge;
      bool real = id != kNoEdge;
      if (real && id >= n) atomicAdd(bad, 1u);
      uint64_t m = ballot(real);
      if (real) ids[deg + lanes_below(m)] = id;
      deg += (uint32_t)__popcll(m);
    }
    for (uint32_t j = deg + l; j < R; j += kWave) ids[j] = kNoEdge;
    if (l == 0) *reinterpret_cast<uint32_t *>(adj) = deg;
  }
}

// ---- medoid -----------------------------------------------------------------
// uint8: exact column sums (any order gives the same integers).  A block takes
// kSumRows rows; thread t sums the dword column t % dw over every
// (256 / dw)-th row, the block adds its partial sums in LDS and then once per
// column in memory.  Bound by the one read of the rows; the first form (one
// thread per byte column, 4,096 rows per block: 74 blocks at 300k rows, one
// byte per load) took 787 us there.
constexpr uint32_t kSumRows = 512;  // 512 * 255 fits 32 bits with room
__global__ __launch_bounds__(256) void column_sums_u8(const uint8_t *x, uint32_t n, uint32_t D,
                                                      unsigned long long *sums) {
  __shared__ uint32_t part[512];
  for (uint32_t d = threadIdx.x; d < D; d += blockDim.x) part[d] = 0;
  __syncthreads();
  const uint32_t dw = D / 4, groups = blockDim.x / dw;  // D <= 512: at least one group
  const uint32_t g = threadIdx.x / dw, c = threadIdx.x % dw;
  const uint32_t r0 = blockIdx.x * kSumRows, r1 = min(n, r0 + kSumRows);
  if (g < groups) {
    const uint32_t *w = reinterpret_cast<const uint32_t *>(x) + c;
    uint32_t s[4] = {0, 0, 0, 0};
#pragma unroll 8
    for (uint32_t i = r0 + g; i < r1; i += groups) {
      const uint32_t v = w[(uint64_t)i * dw];
#pragma unroll
      for (int b = 0; b < 4; ++b) s[b] += (v >> (8 * b)) & 0xFFu;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) atomicAdd(&part[4 * c + b], s[b]);
  }
  __syncthreads();
  for (uint32_t d = threadIdx.x; d < D; d += blockDim.x) atomicAdd(&sums[d], (unsigned long long)part[d]);
}

// float32: column sums in float64 in node order.  The order is part of the
// entry rule, and a serial chain over n rows waits for memory and adder alike
// (1M x 96: 65.4 ms with one thread per column and eight loads in flight), so
// the runs of kSumRun rows are worked out side by side (ordered_sum.hpp): the
// rows are read twice at memory speed, and the chain that is left has one step
// per run (1M x 96: 0.19 ms for the two reads and the starts, 0.57 ms for the chain).
__global__ __launch_bounds__(256) void sum_outlines_f32(const float *x, uint32_t n, uint32_t D, uint32_t runs,
                                                        RunOutline *out) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (uint64_t)runs * D) return;
  const uint32_t c = (uint32_t)(t / D), d = (uint32_t)(t - (uint64_t)c * D);
  const uint32_t r0 = c * kSumRun, rows = min(kSumRun, n - r0);
  const float *p = x + (uint64_t)r0 * D + d;
  RunOutline o = outline_start();
#pragma unroll 16
  for (uint32_t i = 0; i < rows; ++i) outline_add(o, p[(uint64_t)i * D]);
  out[t] = o;
}

// One block per column: the runs' start sums (plain prefix sums, kept in
// place of the outlines' sums, which move to `plain`) and the largest magnitude a partial sum reaches.
__global__ __launch_bounds__(256) void sum_starts_f32(RunOutline *runs_out, double *plain, uint32_t D, uint32_t runs,
                                                      double *most) {
  __shared__ double part[256];
  const uint32_t d = blockIdx.x, t = threadIdx.x;
  const uint32_t each = (runs + 255) / 256, c0 = min(runs, t * each), c1 = min(runs, c0 + each);
  double s = 0.0;
  for (uint32_t c = c0; c < c1; ++c) s += runs_out[(uint64_t)c * D + d].sum;
  part[t] = s;
  __syncthreads();
  if (t == 0) {
    double a = 0.0;
    for (int i = 0; i < 256; ++i) {
      const double v = part[i];
      part[i] = a;
      a += v;
    }
  }
  __syncthreads();
  s = part[t];
  __syncthreads();
  double m = 0.0;
  for (uint32_t c = c0; c < c1; ++c) {
    RunOutline &o = runs_out[(uint64_t)c * D + d];
    const double sum = o.sum, lo = fabs(s + o.lo), hi = fabs(s + o.hi);
    o.sum = s;
    plain[(uint64_t)c * D + d] = sum;
    // (after a NaN every run is open: its start is one)
    m = m >= lo ? m : lo;
    m = m >= hi ? m : hi;
    s += sum;
  }
  part[t] = m;
  __syncthreads();
  if (t == 0) {
    for (int i = 1; i < 256; ++i) m = m >= part[i] ? m : part[i];
    most[d] = m;
  }
}

__global__ __launch_bounds__(256) void sum_amounts_f32(const float *x, uint32_t n, uint32_t D, uint32_t runs,
                                                       const RunOutline *outl, const double *plain, const double *most,
                                                       RunAmount *out) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (uint64_t)runs * D) return;
  const uint32_t c = (uint32_t)(t / D), d = (uint32_t)(t - (uint64_t)c * D);
  const uint32_t r0 = c * kSumRun, rows = min(kSumRun, n - r0);
  const RunOutline o = outl[t];
  const double margin = sum_margin(n, most[d]);
  RunAmount a = run_open(o, margin);
  a.odd = plain[t];
  double even, odd;
  if (o.lo == 0.0 && o.hi == 0.0) {
    // every partial sum 0: all terms are zeros
    a = {0.0, 0.0};
  } else if (run_stand_ins(o.sum, o.lo, o.hi, margin, even, odd)) {
    const float *p = x + (uint64_t)r0 * D + d;
    double s0 = even, s1 = odd;
#pragma unroll 16
    for (uint32_t i = 0; i < rows; ++i) {
      const double v = (double)p[(uint64_t)i * D];
      s0 = __dadd_rn(s0, v);
      s1 = __dadd_rn(s1, v);
    }
    a = {__dsub_rn(s0, even), __dsub_rn(s1, odd)};
  }
  out[t] = a;
}

constexpr uint32_t kSumDirectRuns = 4;

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  return __longlong_as_double((long long)readlane64((uint64_t)__double_as_longlong(v), lane));
}

// One wave per column: 64 runs' amounts are read at once, one per lane, and
// added one after another; an open run's rows likewise.  Without AMOUNTS every
// run is open.
template <bool AMOUNTS>
__global__ __launch_bounds__(kWave) void sum_chain_f32(const float *x, uint32_t n, uint32_t D, uint32_t runs,
                                                       const RunAmount *amounts, double *sums) {
  const uint32_t d = blockIdx.x, l = lane_id();
  double s = 0.0;
  RunAmount next = {sum_open_mark(), 0.0};
  if (AMOUNTS && l < runs) next = amounts[(uint64_t)l * D + d];
  for (uint32_t c0 = 0; c0 < runs; c0 += kWave) {
    const RunAmount a = next;
    const uint32_t cn = c0 + kWave + l;
    if (AMOUNTS && cn < runs) next = amounts[(uint64_t)cn * D + d];
    const uint64_t open = ballot(!(a.even == a.even));
    const uint32_t m = min((uint32_t)kWave, runs - c0);
    for (uint32_t j = 0; j < m; ++j) {
      if (!((open >> j) & 1ull)) {
        const double e = readlane_f64(a.even, (int)j), o = readlane_f64(a.odd, (int)j);
        s = __dadd_rn(s, sum_is_odd(s) ? o : e);
        continue;
      }
      if (run_is_exact(s, readlane_f64(a.even, (int)j))) {
        s = __dadd_rn(s, readlane_f64(a.odd, (int)j));
        continue;
      }
      const uint32_t r0 = (c0 + j) * kSumRun, rows = min(kSumRun, n - r0);
      constexpr int kBlocks = kSumRun / kWave;
      float v[kBlocks];
#pragma unroll
      for (int b = 0; b < kBlocks; ++b) {
        const uint32_t i = b * kWave + l;
        v[b] = i < rows ? x[(uint64_t)(r0 + i) * D + d] : 0.0f;
      }
#pragma unroll
      for (int b = 0; b < kBlocks; ++b) {
        const uint32_t cnt = rows > (uint32_t)b * kWave ? min((uint32_t)kWave, rows - b * kWave) : 0u;
        for (uint32_t i = 0; i < cnt; ++i)
          s = __dadd_rn(s, (double)__uint_as_float(readlane(__float_as_uint(v[b]), (int)i)));
      }
    }
  }
  if (l == 0) sums[d] = s;
}

// key = (distance bits << 32) | id, minimised with one atomic per block.
__device__ __forceinline__ void block_min_key(uint64_t key, unsigned long long *best) {
  __shared__ uint64_t part[256 / kWave];
  for (int m = 1; m < kWave; m <<= 1) key = min64(key, shfl_xor64(key, m));
  if (lane_id() == 0) part[threadIdx.x / kWave] = key;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t b = part[0];
    for (uint32_t w = 1; w < blockDim.x / kWave; ++w) b = min64(b, part[w]);
    atomicMin(best, (unsigned long long)b);
  }
}

__global__ __launch_bounds__(256) void nearest_to_centroid_u8(const uint8_t *x, uint32_t n, uint32_t D,
                                                              const unsigned long long *sums,
                                                              unsigned long long *best) {
  __shared__ uint8_t c[512];
  for (uint32_t d = threadIdx.x; d < D; d += blockDim.x)
    c[d] = (uint8_t)((sums[d] + n / 2) / n);
  __syncthreads();
  uint64_t key = kInfKey;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    uint32_t s = 0;
    for (uint32_t d = 0; d < D; ++d) {
      int t = (int)c[d] - (int)x[(uint64_t)i * D + d];
      s += (uint32_t)(t * t);
    }
    key = min64(key, ((uint64_t)s << 32) | i);
  }
  block_min_key(key, best);
}

__global__ __launch_bounds__(256) void nearest_to_centroid_f32(const float *x, uint32_t n, uint32_t D,
                                                               const double *sums,
                                                               unsigned long long *best) {
  __shared__ float c[256];
  for (uint32_t d = threadIdx.x; d < D; d += blockDim.x) c[d] = (float)(sums[d] / (double)n);
  __syncthreads();
  uint64_t key = kInfKey;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    float acc = 0.0f;
    for (uint32_t d = 0; d < D; ++d) {
      float t = __fsub_rn(c[d], x[(uint64_t)i * D + d]);
      acc = __fadd_rn(acc, __fmul_rn(t, t));
    }
    key = min64(key, ((uint64_t)__float_as_uint(acc) << 32) | i);
  }
  block_min_key(key, best);
}

}  // namespace gorio
