// Cluster placement and query ordering for paged search (host entry points
// and their kernels).
//
// Pages are the unit of remote I/O (GORIO Sec. 3.1), so which nodes share a
// page, and which queries run at the same time, decide how often a fetched
// page is used again before the clock hand evicts it.  The disk-resident ANNS
// work the paper builds on studies page layout and graph locality (Sec. 6);
// the paper's future work asks for miss coalescing across queries (Sec. 7.2).
// Here: a few Lloyd iterations of k-means on the GPU give K centroids; nodes
// are placed cluster by cluster (node_to_slot), and a paged search admits its
// queries cluster by cluster, so the queries in flight at any time read a
// small set of clusters' pages, which the cache then holds.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "../../include/gorio.h"
#include "cluster.hpp"
#include "cluster_kernels.hpp"

namespace gorio {
gorio_status fail(gorio_status st, const char *fmt, ...);

template <typename T>
hipError_t launch_nearest_centroid_t(const T *v, uint64_t count, uint32_t D, const float *c, const float *cc,
                                     uint32_t K, uint32_t *out, hipStream_t s) {
  const int block = 256;
  const unsigned grid = (unsigned)((count + block - 1) / block);
  switch (D) {
    case 32: nearest_centroid<T, 32><<<grid, block, 0, s>>>(v, count, D, c, cc, K, out); break;
    case 64: nearest_centroid<T, 64><<<grid, block, 0, s>>>(v, count, D, c, cc, K, out); break;
    case 96: nearest_centroid<T, 96><<<grid, block, 0, s>>>(v, count, D, c, cc, K, out); break;
    case 128: nearest_centroid<T, 128><<<grid, block, 0, s>>>(v, count, D, c, cc, K, out); break;
    default: nearest_centroid<T, 0><<<grid, block, 0, s>>>(v, count, D, c, cc, K, out); break;
  }
  return hipGetLastError();
}

hipError_t launch_nearest_centroid(gorio_dtype dt, const void *v, uint64_t count, uint32_t D, const float *c,
                                   const float *cc, uint32_t K, uint32_t *out, hipStream_t s) {
  if (count == 0) return hipSuccess;
  if (dt == GORIO_U8)
    return launch_nearest_centroid_t(static_cast<const uint8_t *>(v), count, D, c, cc, K, out, s);
  return launch_nearest_centroid_t(static_cast<const float *>(v), count, D, c, cc, K, out, s);
}

namespace {

// Device memory of one gorio_cluster_order call.
struct ClusterWork {
  uint32_t Kp, DP;         // centroids and dimensions, padded for the matrix path
  float *c;                // K x D
  float *rows, *cols, *cc; // centroid_layouts' outputs
  uint64_t *hash;
  unsigned int *flags;     // [pairs, open vectors, largest norm's bits]
  uint32_t *key, *alt, *pairs, *open;
};

// The matrix path takes whole batches: below these sizes (no wave for every
// SIMD, or tiles mostly padding) the plain kernel is as fast, and its register
// arrays end at 256 dimensions.
bool matrix_path(uint64_t count, uint32_t D, uint32_t K) { return D <= 256 && K >= 32 && count >= 16384; }
uint32_t padded_dims(uint32_t D) { return D <= 32 ? 32 : D <= 64 ? 64 : D <= 96 ? 96 : D <= 128 ? 128 : D <= 192 ? 192 : 256; }

template <typename T, int DQ, int NT>
void launch_matrix(const T *v, uint64_t n, uint32_t D, const ClusterWork &w, hipStream_t s) {
  const unsigned grid = (unsigned)((n + 128 * NT - 1) / (128 * NT));
  nearest_matrix<T, DQ, NT><<<grid, 256, 0, s>>>(v, n, D, w.rows, w.cc, w.Kp, w.flags + 2, w.key, w.alt, w.pairs,
                                                 w.open, w.flags);
}

// w.key = nearest centroid of every vector.
template <typename T>
hipError_t assign(const T *v, uint64_t n, uint32_t D, uint32_t K, const ClusterWork &w, hipStream_t s) {
  fill_words<<<1, 64, 0, s>>>(w.flags, 4, 0u);
  centroid_layouts<<<(w.Kp + 63) / 64, 64, 0, s>>>(w.c, K, D, w.DP, w.Kp, w.rows, w.cols, w.cc, w.hash,
                                                  w.flags + 2);
  if (!matrix_path(n, D, K)) return launch_nearest_centroid_t(v, n, D, w.c, w.cc, K, w.key, s);
  drop_repeats<<<K, kWave, 0, s>>>(w.c, D, w.hash, w.cc);
  switch (w.DP) {
    case 32: launch_matrix<T, 4, 2>(v, n, D, w, s); break;
    case 64: launch_matrix<T, 8, 2>(v, n, D, w, s); break;
    case 96: launch_matrix<T, 12, 2>(v, n, D, w, s); break;
    case 128: launch_matrix<T, 16, 2>(v, n, D, w, s); break;
    case 192: launch_matrix<T, 24, 1>(v, n, D, w, s); break;
    default: launch_matrix<T, 32, 1>(v, n, D, w, s); break;
  }
  nearest_of_pair<T><<<1024, 256, 0, s>>>(v, D, w.c, w.cc, w.pairs, w.flags, w.alt, w.key);
  nearest_of_all<T><<<2048, kWave, 0, s>>>(v, D, w.cols, w.cc, K, w.Kp, w.open, w.flags + 1, w.key);
  return hipGetLastError();
}

// w.c = means of the clusters' members.  uint8: sums of K x D whole numbers;
// float32: kMeanRanges x K x D float64.
void update_means(const uint8_t *v, uint64_t n, uint32_t D, uint32_t K, const ClusterWork &w, const uint32_t *order,
                  const uint32_t *start, void *sums, hipStream_t s) {
  auto *whole = static_cast<unsigned long long *>(sums);
  const uint64_t cells = (uint64_t)K * D;
  fill_words<<<(unsigned)std::min<uint64_t>(4096, (2 * cells + 255) / 256), 256, 0, s>>>(
      static_cast<uint32_t *>(sums), 2 * cells, 0u);
  const uint32_t rows = sum_rows_u8(n);
  const unsigned grid = (unsigned)((n + rows - 1) / rows);
  if (D % 4 == 0) cluster_sums_u8<4><<<grid, 256, 0, s>>>(v, (uint32_t)n, D, rows, order, w.key, start, whole);
  else cluster_sums_u8<1><<<grid, 256, 0, s>>>(v, (uint32_t)n, D, rows, order, w.key, start, whole);
  cluster_means_u8<<<(unsigned)((cells + 255) / 256), 256, 0, s>>>(whole, start, K, D, w.c);
}
void update_means(const float *v, uint64_t n, uint32_t D, uint32_t K, const ClusterWork &w, const uint32_t *order,
                  const uint32_t *start, void *sums, hipStream_t s) {
  const uint64_t cells = (uint64_t)K * D;
  cluster_sums_f32<<<kMeanRanges * K, std::min(256u, (D + 63) / 64 * 64), 0, s>>>(v, n, D, order, start,
                                                                                 static_cast<double *>(sums));
  cluster_means_f32<<<(unsigned)((cells + 255) / 256), 256, 0, s>>>(static_cast<double *>(sums), start, K, D, w.c);
}

}  // namespace

void centroid_norms(const float *c, uint32_t K, uint32_t D, float *cc) {
  for (uint32_t k = 0; k < K; ++k) {
    float s = 0.0f;
    for (uint32_t d = 0; d < D; ++d) s += c[(uint64_t)k * D + d] * c[(uint64_t)k * D + d];
    cc[k] = s;
  }
}

void order_by_key(const uint32_t *key, uint64_t count, uint32_t K, uint32_t *order) {
  std::vector<uint64_t> start(K + 1, 0);
  for (uint64_t i = 0; i < count; ++i) ++start[key[i] + 1];
  for (uint32_t k = 0; k < K; ++k) start[k + 1] += start[k];
  for (uint64_t i = 0; i < count; ++i) order[start[key[i]]++] = (uint32_t)i;
}

}  // namespace gorio

using namespace gorio;

#define HIP_OR_FAIL(expr)                                                                  \
  do {                                                                                     \
    hipError_t e_ = (expr);                                                                \
    if (e_ != hipSuccess)                                                                  \
      return fail(e_ == hipErrorOutOfMemory ? GORIO_ENOMEM : GORIO_EDEVICE, "%s: %s", #expr, \
                  hipGetErrorString(e_));                                                  \
  } while (0)

namespace {
struct Buf {
  void *p = nullptr;
  ~Buf() { if (p) (void)hipFree(p); }
  hipError_t alloc(size_t bytes) { return hipMalloc(&p, bytes ? bytes : 4); }
};
struct StreamGuard {
  hipStream_t s = nullptr;
  ~StreamGuard() { if (s) (void)hipStreamDestroy(s); }
};
}  // namespace

extern "C" gorio_status gorio_cluster_order(gorio_dtype dtype, const void *vectors, uint64_t n, uint32_t D,
                                            uint32_t clusters, uint32_t iterations, uint32_t *node_to_slot,
                                            float *centroids) {
  if (!vectors || !node_to_slot || !centroids) return fail(GORIO_EINVAL, "vectors, node_to_slot and centroids must be non-NULL");
  if (dtype != GORIO_U8 && dtype != GORIO_F32) return fail(GORIO_EINVAL, "unknown dtype %d", (int)dtype);
  if (n == 0 || n >= (1ull << 31)) return fail(GORIO_EINVAL, "n=%llu outside [1, 2^31)", (unsigned long long)n);
  if (D == 0 || D > 1024) return fail(GORIO_EINVAL, "D=%u outside [1, 1024]", D);
  if (clusters == 0 || clusters > kMaxClusters || clusters > n)
    return fail(GORIO_EINVAL, "clusters=%u outside [1, min(n, %u)]", clusters, kMaxClusters);
  if (iterations > 64) return fail(GORIO_EINVAL, "iterations=%u above 64", iterations);
  const uint32_t K = clusters, N = (uint32_t)n;
  const size_t eb = dtype == GORIO_U8 ? 1 : 4;
  StreamGuard sg;
  HIP_OR_FAIL(hipStreamCreateWithFlags(&sg.s, hipStreamNonBlocking));
  hipStream_t s = sg.s;
  ClusterWork w;
  w.Kp = (K + 31) / 32 * 32;
  w.DP = D <= 256 ? padded_dims(D) : D;
  // tiles of the counting sort: 2,048 nodes (32 steps of a wave), more when
  // many clusters would make the table of counts large
  uint32_t tile = 2048;
  while ((uint64_t)((N + tile - 1) / tile) * K > (1ull << 26) && tile < (1u << 30)) tile *= 2;
  const uint32_t tiles = (N + tile - 1) / tile;
  uint32_t key_bits = 0;
  while ((1ull << key_bits) < K) ++key_bits;

  size_t bytes = 0;
  auto take = [&](size_t b) {
    const size_t at = bytes;
    bytes += (b + 255) & ~(size_t)255;
    return at;
  };
  const size_t o_v = take(n * D * eb), o_c = take((size_t)K * D * 4), o_rows = take((size_t)w.Kp * w.DP * 4),
               o_cols = take((size_t)w.Kp * D * 4), o_cc = take((size_t)w.Kp * 4), o_hash = take((size_t)w.Kp * 8),
               o_flags = take(16),
               o_key = take(n * 4), o_alt = take(n * 4), o_pairs = take(n * 4), o_open = take(n * 4),
               o_slot = take(n * 4), o_hist = take((size_t)tiles * K * 4), o_total = take((size_t)K * 4),
               o_start = take((size_t)(K + 1) * 4),
               o_sums = take(iterations ? (dtype == GORIO_U8 ? 1 : kMeanRanges) * (size_t)K * D * 8 : 0);
  Buf work;
  HIP_OR_FAIL(work.alloc(bytes));
  uint8_t *base = static_cast<uint8_t *>(work.p);
  auto words = [&](size_t at) { return reinterpret_cast<uint32_t *>(base + at); };
  auto floats = [&](size_t at) { return reinterpret_cast<float *>(base + at); };
  w.c = floats(o_c);
  w.rows = floats(o_rows);
  w.cols = floats(o_cols);
  w.cc = floats(o_cc);
  w.hash = reinterpret_cast<uint64_t *>(base + o_hash);
  w.flags = words(o_flags);
  w.key = words(o_key);
  w.alt = words(o_alt);
  w.pairs = words(o_pairs);
  w.open = words(o_open);
  uint32_t *slot = words(o_slot), *order = w.alt, *rank = w.pairs;  // the lists are done with by then
  uint32_t *hist = words(o_hist), *total = words(o_total), *start = words(o_start);
  const uint8_t *v8 = base + o_v;
  const float *vf = floats(o_v);
  HIP_OR_FAIL(hipMemcpyAsync(base + o_v, vectors, n * D * eb, hipMemcpyHostToDevice, s));

  // initial centroids: the vectors of nodes i * n / K (distinct ids)
  std::vector<float> c((size_t)K * D);
  for (uint32_t k = 0; k < K; ++k) {
    const uint64_t i = (uint64_t)k * n / K;
    for (uint32_t d = 0; d < D; ++d)
      c[(size_t)k * D + d] = dtype == GORIO_U8 ? (float)static_cast<const uint8_t *>(vectors)[i * D + d]
                                               : static_cast<const float *>(vectors)[i * D + d];
  }
  HIP_OR_FAIL(hipMemcpyAsync(w.c, c.data(), c.size() * 4, hipMemcpyHostToDevice, s));

  // Lloyd iterations, then the placement: cluster by cluster, id order inside
  // a cluster.  Nothing returns to the host in between.
  for (uint32_t it = 0;; ++it) {
    HIP_OR_FAIL(dtype == GORIO_U8 ? assign(v8, n, D, K, w, s) : assign(vf, n, D, K, w, s));
    const uint64_t cells = (uint64_t)tiles * K;
    fill_words<<<(unsigned)std::min<uint64_t>(4096, (cells + 255) / 256), 256, 0, s>>>(hist, cells, 0u);
    tile_ranks<<<tiles, kWave, 0, s>>>(w.key, N, K, key_bits, tile, hist, rank);
    tile_prefix<<<(K + 63) / 64, 64, 0, s>>>(hist, tiles, K, total);
    cluster_starts<<<1, 1024, 0, s>>>(total, K, start);
    cluster_slots<<<(N + 255) / 256, 256, 0, s>>>(w.key, rank, hist, start, N, K, tile, slot, order);
    HIP_OR_FAIL(hipGetLastError());
    if (it == iterations) break;
    // each centroid becomes the mean of its members (an empty cluster keeps
    // its centroid)
    if (dtype == GORIO_U8) update_means(v8, n, D, K, w, order, start, base + o_sums, s);
    else update_means(vf, n, D, K, w, order, start, base + o_sums, s);
    HIP_OR_FAIL(hipGetLastError());
  }
  HIP_OR_FAIL(hipMemcpyAsync(c.data(), w.c, c.size() * 4, hipMemcpyDeviceToHost, s));
  HIP_OR_FAIL(hipMemcpyAsync(node_to_slot, slot, n * 4, hipMemcpyDeviceToHost, s));
  HIP_OR_FAIL(hipStreamSynchronize(s));
  memcpy(centroids, c.data(), c.size() * 4);
  return GORIO_OK;
}
