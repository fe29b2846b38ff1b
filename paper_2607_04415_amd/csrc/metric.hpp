// Distance policies of the search kernels (squared L2, returned squared).
//
// A policy loads the query, evaluates the entry node, and turns a batch of
// candidate records into 64-bit frontier keys (distance bits << 32 |
// id << 1).  The kernels' traversal, filtering and merging do not depend on
// the element type: uint8 distances are non-negative int32 values and float32
// distances are >= +0, so both order correctly as unsigned 32-bit patterns.
//
//   MetricU8  - exact int32 distance: q.q + sum (x.x - 2 q.x) with
//               v_dot4_u32_u8 on coalesced reads, 8 lanes per vector.
//   MetricU8Rows - the same for rows of other lengths, arrangements and
//               placements (resident).
//   MetricF32, MetricF32Lines, MetricF32Own - one lane per candidate (the
//               resident kernel gathers 8 lanes per vector by whole lines and
//               hands the blocks to their lanes through LDS; rows of up to 8
//               floats are read by their own lane);
//               t = q_d - x_d, acc = acc + t*t for d = 0 .. D-1 in order,
//               every operation rounded to nearest even with no fused
//               multiply-add, so the result is the same float as a plain
//               sequential loop.
#pragma once

#include "frontier.hpp"
#include "page_cache.hpp"

namespace gorio {

// ---------------------------------------------------------------------------
// uint8
// ---------------------------------------------------------------------------
// LOC16: the kernel keeps each candidate as its vector's 16-byte locator
// (identity placement, units16 != 0) instead of its id, stored so that the
// kRounds candidates of each group of 8 lanes are consecutive words: the
// batch's addresses arrive with kRounds / 4 LDS reads and no per-round
// address arithmetic, and ids are recovered from locators for the keys.
template <int VDW, bool EXACT, bool LOC16 = false>
struct MetricU8 {
  // vectors in flight per resident gather batch: 128 for up to 16 B per lane,
  // 64 for wider rows (kept small so that two waves fit each SIMD's registers)
  static constexpr int kRounds = VDW <= 4 ? 16 : 8;
  static constexpr int kBatch = kRounds * 8;
  static constexpr int kChunks = kBatch / kWave;
  static_assert(kRounds % 8 == 0, "rounds are reduced eight at a time");
  static constexpr int kQueryWords = 1;          // the query lives in registers
  // resident kernel: waves per SIMD that its registers leave room for, those of
  // the grid, and the 16-bit visited table.  Frontiers of up to 64: 4096 entries in 8 KB and
  // 128 registers; the grid holds two waves per SIMD, which keep the gathers
  // saturated (a 100k-query batch on the 1M x 128-d index runs at the same
  // rate with two or four per SIMD) while each query, and so a batch's tail,
  // finishes sooner (10k queries: 0.79 ms against 0.85 ms with four).  Longer
  // frontiers meet more nodes than 4096 entries record (L=128, W=8, R=64: 80M
  // of 148M evaluations were repeats), and two waves per SIMD leave room for
  // 16 KB each.  Their kernels are still scheduled for four: the schedule for
  // two is 2 to 4% slower (100k nodes, R=16, 5,000 queries, us a call: 128
  // bytes, L=128 449 for two and 441 for four; 32 bytes, L=200 834 and 814;
  // 16 bytes, L=200 755 and 732), but for locators with four frontier
  // registers, which do not fit 128 (L=200 735 and 804).
  __host__ __device__ static constexpr int waves_per_simd(int kpl, uint32_t) {
    return VDW <= 4 && !(LOC16 && kpl > 2) ? 4 : 2;
  }
  __host__ __device__ static constexpr int grid_waves_per_simd(int, uint32_t table_words) {
    return table_words > 4096 ? 1 : 2;
  }
  __host__ __device__ static constexpr int ht_log2(int kpl) { return VDW <= 4 && kpl == 1 ? 12 : 13; }
  __host__ __device__ static constexpr int few_ht_log2(int kpl) { return ht_log2(kpl); }
  static constexpr uint32_t kPadDist = 0x7FFFFFFFu;  // INT32_MAX
  static_assert(!LOC16 || (EXACT && VDW % 4 == 0), "locators address whole 16-byte units");
  static constexpr bool kLocators = LOC16;
  static constexpr bool kStream = LOC16;    // chunks of 64, two in flight
  static constexpr bool kOffsets = false;   // candidates' byte offsets kept in LDS
  __host__ __device__ static constexpr uint32_t stage_words(int, uint32_t) { return 0; }  // LDS of a wave for set_stage
  // search_team (locators): waves per query, per SIMD at least, visited table
  __host__ __device__ static constexpr int team_waves(int kpl) { return kpl > 1 ? 8 : 4; }
  __host__ __device__ static constexpr int team_per_simd() { return 2; }
  __host__ __device__ static constexpr int team_ht_log2(int) { return 13; }
  static constexpr int kTeamStageWords = 0;
  __device__ __forceinline__ void set_stage(uint32_t *) {}
  static constexpr bool kGathered = false;  // float32 line gather only

  // Where the kernel's compaction puts the i-th new candidate, and the word
  // it stores for node v (its id, or with LOC16 its vector's locator).
  __device__ __forceinline__ static uint32_t cand_pos(uint32_t i) {
    if constexpr (LOC16)
      return (i & ~(uint32_t)(kBatch - 1)) | ((i & 7u) * kRounds) | ((i >> 3) & (uint32_t)(kRounds - 1));
    else
      return i;
  }
  __device__ __forceinline__ static uint32_t cand_word(const PageGeom &geom, uint32_t v) {
    if constexpr (LOC16) return vec_locator(geom, v);
    else return v;
  }

  // After compaction of cnt candidates: give the rest of the last chunk of 64
  // the fallback node's word, so that every lane of every round of a chunk
  // loads a vector (the chunk's load count is then fixed).
  __device__ __forceinline__ static void pad_round(uint32_t *cand, uint64_t *, uint32_t cnt, uint32_t fallback_word,
                                                   uint64_t) {
    if constexpr (LOC16) {
      const uint32_t i = cnt + (uint32_t)lane_id();
      if (i < ((cnt + kWave - 1) & ~(uint32_t)(kWave - 1))) cand[cand_pos(i)] = fallback_word;
    }
  }

  U8Vec<VDW, EXACT> q;
  int qq;
  uint32_t dwords;

  __device__ __forceinline__ void load_query(const void *queries, uint32_t qi, uint32_t D, uint32_t *) {
    const int gl = lane_id() & 7;
    dwords = D >> 2;
    q.load(static_cast<const uint8_t *>(queries) + (uint64_t)qi * D, gl, dwords);
    int s = 0;
#pragma unroll
    for (int t = 0; t < VDW; ++t) s += (int)__builtin_amdgcn_udot4(q.w[t], q.w[t], 0u, false);
    qq = sum8(s);
  }

  // Distance bits of one record, computed by the whole wave (uniform result).
  __device__ __forceinline__ uint32_t dist_one(const uint8_t *pages, uint64_t off) const {
    const uint8_t *rec = pages + off;
    U8Vec<VDW, EXACT> x;
    x.load(rec, lane_id() & 7, dwords);
    return (uint32_t)(sum8(partial_u8(q, x)) + qq);
  }

  // Keys of candidates c0 .. c0 + kBatch - 1 of cand (kInfKey past cnt), from
  // the resident pages.  One round trip for the batch.
  template <bool N2S>
  __device__ __forceinline__ void resident_keys(const uint8_t *pages, const PageGeom &geom, const uint32_t *cand,
                                                uint32_t c0, uint32_t cnt, uint32_t fallback,
                                                uint64_t (&key)[kChunks]) const {
    static_assert(!LOC16, "with locators the kernel streams chunks (chunk_issue, chunk_key)");
    const int l = lane_id();
    const int g = l >> 3;
    const int gl = l & 7;
    // candidate node -> record; lanes past the count read the fallback record
    uint64_t rec[kRounds];
#pragma unroll
    for (int rr = 0; rr < kRounds; ++rr) {
      if (c0 + rr * 8 >= cnt) break;
      const uint32_t idx = c0 + rr * 8 + g;
      rec[rr] = vec_offset(geom, slot_ct<N2S>(geom, idx < cnt ? cand[idx] : fallback));
    }
    U8Vec<VDW, EXACT> x[kRounds];
#pragma unroll
    for (int rr = 0; rr < kRounds; ++rr) {
      if (c0 + rr * 8 >= cnt) break;
      x[rr].load(pages + rec[rr], gl, dwords);
    }
    // eight rounds at a time: lane gl of group g ends with round 8c + gl's distance
    int dist[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      dist[c] = 0;
      if (c0 + c * kWave >= cnt) break;
      int part[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) part[j] = c0 + (c * 8 + j) * 8 < cnt ? partial_u8(q, x[c * 8 + j]) : 0;
      dist[c] = transpose_sum8(part) + qq;
    }
    // lane l of chunk c holds candidate c0 + 64c + 8*(l%8) + l/8
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const uint32_t my_idx = c0 + c * kWave + gl * 8 + g;
      key[c] = my_idx < cnt ? (((uint64_t)(uint32_t)dist[c] << 32) | ((uint64_t)cand[my_idx] << 1)) : kInfKey;
    }
  }

  // Streaming gather (LOC16): the candidate list is evaluated in chunks of
  // 64, eight rounds of eight vectors; the kernel keeps two chunks in flight
  // (issues the next while reducing and merging the current one).  Group g's
  // eight locators of chunk c0 / 64 are consecutive words of the compacted
  // list (cand_pos).  Every chunk issues the same number of loads, so the
  // compiler's waits before a chunk's use leave the other chunk in flight.
  struct Chunk {
    U8Vec<VDW, EXACT> x[8];
  };
  __device__ __forceinline__ void chunk_issue(const uint8_t *pages, const PageGeom &geom, const uint32_t *cand,
                                              const uint64_t *, uint32_t c0, Chunk &ck) const {
    const __amdgpu_buffer_rsrc_t rs = units16_rsrc(pages, geom);
    static_assert(LOC16 && kRounds == 16, "streaming needs locators and 16 rounds per 128 candidates");
    const int l = lane_id();
    const int g = l >> 3;
    const int gl = l & 7;
    const uint4 *src = reinterpret_cast<const uint4 *>(cand + (c0 & ~127u) + g * kRounds + ((c0 >> 6) & 1u) * 8u);
    const uint4 a = src[0], b = src[1];
    uint32_t loc[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) asm volatile("" : "+v"(loc[rr]));
    // all eight rounds: positions past the count hold the fallback's locator
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) {
      const uint32_t u = loc[rr] + (uint32_t)gl * (VDW / 4);
#pragma unroll
      for (int t = 0; t < VDW; t += 4) {
        const u32x4_t v = struct_buffer_load_b128(rs, (int)(u + t / 4), 0, 0, 0);
        ck.x[rr].w[t] = v.x; ck.x[rr].w[t + 1] = v.y; ck.x[rr].w[t + 2] = v.z; ck.x[rr].w[t + 3] = v.w;
      }
    }
  }
  // Key of this lane's candidate of the chunk (kInfKey past cnt): lane
  // (g, gl) ends with round gl of group g, candidate c0 + 8 gl + g.
  __device__ __forceinline__ uint64_t chunk_key(const PageGeom &geom, const uint32_t *cand, uint32_t c0,
                                                uint32_t cnt, const Chunk &ck) const {
    const int l = lane_id();
    const int g = l >> 3;
    const int gl = l & 7;
    int part[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) part[j] = partial_u8(q, ck.x[j]);
    const int dist = transpose_sum8(part) + qq;
    const bool ok = c0 + (uint32_t)gl * 8 + (uint32_t)g < cnt;
    const uint32_t pos = (c0 & ~127u) + g * kRounds + ((c0 >> 6) & 1u) * 8u + gl;
    const uint32_t v = ok ? slot_of_locator(geom, cand[pos]) : 0u;
    return ok ? (((uint64_t)(uint32_t)dist << 32) | ((uint64_t)v << 1)) : kInfKey;
  }

  // Paged: keys of the candidates whose pages are ready (rdy, slot per lane;
  // candidate index = base + lane).  off_of(slot, node) is the record's byte
  // offset in the cache.  The ready lanes are compacted and evaluated 8 per
  // round; the key of the i-th ready candidate ends up in some lane, the others
  // hold kInfKey.
  template <class OffOf>
  __device__ __forceinline__ uint64_t paged_keys(OffOf off_of, __amdgpu_buffer_rsrc_t crs, const uint32_t *cand,
                                                 uint32_t base, bool rdy, uint32_t slot, uint64_t mr) const {
    const int l = lane_id();
    const int g = l >> 3;
    const int gl = l & 7;
    const uint32_t cnt = (uint32_t)__popcll(mr);
    __shared__ uint32_t rc[kWave], rs[kWave];
    if (rdy) {
      const uint32_t my_rank = lanes_below(mr);
      rc[my_rank] = base + l;
      rs[my_rank] = slot;
    }
    __syncthreads();
    U8Vec<VDW, EXACT> x[8];
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) {
      const uint32_t idx = rr * 8 + g;
      const uint32_t ci = idx < cnt ? rc[idx] : rc[0];
      const uint32_t si = idx < cnt ? rs[idx] : rs[0];
      load_cached_u8(x[rr], crs, off_of(si, cand[ci]), gl);
    }
    int part[8];
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) part[rr] = partial_u8(q, x[rr]);
    const int mine_d = transpose_sum8(part) + qq;
    const uint32_t my_idx = gl * 8 + g;
    uint64_t key = kInfKey;
    if (my_idx < cnt) key = ((uint64_t)(uint32_t)mine_d << 32) | ((uint64_t)cand[rc[my_idx]] << 1);
    __syncthreads();
    return key;
  }

 private:
  // coherent read of a cached vector (see page_cache.hpp)
  __device__ __forceinline__ void load_cached_u8(U8Vec<VDW, EXACT> &x, __amdgpu_buffer_rsrc_t r, uint32_t rec,
                                                 int gl) const {
    const uint32_t b = rec + (uint32_t)gl * VDW * 4u;
    if constexpr (EXACT && VDW % 4 == 0) {
#pragma unroll
      for (int t = 0; t < VDW; t += 4) {
        const uint4 u = coherent_load_u128(r, b + t * 4u);
        x.w[t] = u.x; x.w[t + 1] = u.y; x.w[t + 2] = u.z; x.w[t + 3] = u.w;
      }
    } else {
#pragma unroll
      for (int t = 0; t < VDW; ++t)
        x.w[t] = (EXACT || (uint32_t)(gl * VDW + t) < dwords) ? coherent_load_u32(r, b + t * 4u) : 0u;
    }
  }
};

// ---------------------------------------------------------------------------
// uint8 rows of any length from 16 bytes up, any arrangement and placement
// (resident kernel; identity-placed 128-byte rows on line starts are MetricU8
// with locators).  8 lanes per vector; lane gl holds the 16-byte units
// gl + 8 t, so each load instruction reads whole lines.  The last unit of a
// ragged row starts 16 bytes before the row's end and masks the bytes that the
// unit before it has already, so nothing past the row is read and every
// dimension counts once.  Candidates' byte offsets are worked out once, when
// they are compacted, and read back from LDS; two chunks of 64 vectors are in
// flight.  Bound by the lines read (a 100-byte row in a 296-byte record lies
// on 1.8 of them).  Against dword loads with a bound check on each, and the
// placement looked up between compaction and gather (300k rows, 5,000 queries,
// L=64, us a launch): 100 bytes, contiguous, placed 620 -> 513; whole calls:
// 128 placed 552 -> 413, 128 contiguous 635 -> 564, 200 bytes 1,319 -> 743, 256
// placed at L=128 2,089 -> 704.
// ---------------------------------------------------------------------------
template <int NU, bool EXACT>
struct MetricU8Rows {
  static constexpr int kQueryWords = 1;
  // two waves per SIMD: 256 registers, 16 KB visited table
  __host__ __device__ static constexpr int waves_per_simd(int, uint32_t) { return 2; }
  __host__ __device__ static constexpr int grid_waves_per_simd(int, uint32_t table_words) {
    return table_words > 4096 ? 1 : 2;
  }
  __host__ __device__ static constexpr int ht_log2(int) { return 13; }
  __host__ __device__ static constexpr int few_ht_log2(int kpl) { return ht_log2(kpl); }
  static constexpr uint32_t kPadDist = 0x7FFFFFFFu;
  static constexpr bool kLocators = false, kGathered = false, kStream = true, kOffsets = true;
  __host__ __device__ static constexpr uint32_t stage_words(int, uint32_t) { return 0; }
  __host__ __device__ static constexpr int team_waves(int kpl) { return kpl > 1 ? 8 : 4; }
  __host__ __device__ static constexpr int team_per_simd() { return 2; }
  __host__ __device__ static constexpr int team_ht_log2(int) { return 13; }
  static constexpr int kTeamStageWords = 0;
  __device__ __forceinline__ void set_stage(uint32_t *) {}

  __device__ __forceinline__ static uint32_t cand_pos(uint32_t i) { return i; }
  __device__ __forceinline__ static uint32_t cand_word(const PageGeom &, uint32_t v) { return v; }
  // the rest of the last chunk reads the fallback vector
  __device__ __forceinline__ static void pad_round(uint32_t *, uint64_t *coff, uint32_t cnt, uint32_t,
                                                   uint64_t fallback_off) {
    const uint32_t i = cnt + (uint32_t)lane_id();
    if (i < ((cnt + kWave - 1) & ~(uint32_t)(kWave - 1))) coff[i] = fallback_off;
  }

  uint32_t q[NU * 4], mask[EXACT ? 1 : NU * 4];
  uint32_t start[NU];  // byte offset of unit t in a row
  int qq;

  struct Row {
    uint32_t w[NU * 4];
  };
  __device__ __forceinline__ void load_row(const uint8_t *row, Row &x) const {
#pragma unroll
    for (int t = 0; t < NU; ++t) {
      uint4 u;
      __builtin_memcpy(&u, __builtin_assume_aligned(row + start[t], 4), 16);
      x.w[4 * t] = u.x; x.w[4 * t + 1] = u.y; x.w[4 * t + 2] = u.z; x.w[4 * t + 3] = u.w;
    }
  }
  __device__ __forceinline__ void load_query(const void *queries, uint32_t qi, uint32_t D, uint32_t *) {
    const uint32_t gl = lane_id() & 7;
#pragma unroll
    for (int t = 0; t < NU; ++t) {
      const uint32_t at = 16u * (gl + 8u * t);
      start[t] = EXACT ? at : min(at, D - 16u);
      if constexpr (!EXACT) {
#pragma unroll
        for (int j = 0; j < 4; ++j) mask[4 * t + j] = at < D && start[t] + 4u * j >= at ? 0xFFFFFFFFu : 0u;
      }
    }
    Row x;
    load_row(static_cast<const uint8_t *>(queries) + (uint64_t)qi * D, x);
    int s = 0;
#pragma unroll
    for (int t = 0; t < NU * 4; ++t) {
      q[t] = EXACT ? x.w[t] : x.w[t] & mask[t];
      s += (int)__builtin_amdgcn_udot4(q[t], q[t], 0u, false);
    }
    qq = sum8(s);
  }
  __device__ __forceinline__ int partial(const Row &x) const {
    uint32_t xx = 0, qx = 0;
#pragma unroll
    for (int t = 0; t < NU * 4; ++t) {
      const uint32_t w = EXACT ? x.w[t] : x.w[t] & mask[t];
      xx = __builtin_amdgcn_udot4(w, w, xx, false);
      qx = __builtin_amdgcn_udot4(q[t], w, qx, false);
    }
    return (int)xx - 2 * (int)qx;
  }
  __device__ __forceinline__ uint32_t dist_one(const uint8_t *pages, uint64_t off) const {
    Row x;
    load_row(pages + off, x);
    return (uint32_t)(sum8(partial(x)) + qq);
  }

  // Group g reads candidates c0 + 8 g .. + 7, so lane l ends with candidate
  // c0 + l.
  struct Chunk {
    Row x[8];
  };
  __device__ __forceinline__ void chunk_issue(const uint8_t *pages, const PageGeom &, const uint32_t *,
                                              const uint64_t *coff, uint32_t c0, Chunk &ck) const {
    const uint64_t *o = coff + c0 + (lane_id() & ~7);
#pragma unroll
    for (int r = 0; r < 8; ++r) load_row(pages + o[r], ck.x[r]);
  }
  __device__ __forceinline__ uint64_t chunk_key(const PageGeom &, const uint32_t *cand, uint32_t c0, uint32_t cnt,
                                                const Chunk &ck) const {
    int part[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) part[r] = partial(ck.x[r]);
    const int dist = transpose_sum8(part) + qq;
    const uint32_t i = c0 + lane_id();
    return i < cnt ? (((uint64_t)(uint32_t)dist << 32) | ((uint64_t)cand[i] << 1)) : kInfKey;
  }
};

// ---------------------------------------------------------------------------
// float32
// ---------------------------------------------------------------------------
// NV4: the vector has at most 4 * NV4 floats.  EXACT: exactly 4 * NV4, read
// with 16-B loads all at once; otherwise dword loads of d < D, 16 at a time.
template <int NV4, bool EXACT>
struct MetricF32 {  // paged kernels: one lane per candidate, records in the page cache
  static constexpr int kQueryWords = 4 * NV4;
  static constexpr uint32_t kPadDist = 0x7F800000u;  // +inf
  static constexpr int kStep = 16;                   // dwords per round trip (generic path)

  const float *qs;  // the query in LDS (wave-uniform reads)
  uint32_t D;

  // Copies the query into LDS; the caller synchronizes before use.
  __device__ __forceinline__ void load_query(const void *queries, uint32_t qi, uint32_t D_, uint32_t *qlds) {
    D = D_;
    const uint32_t *src = static_cast<const uint32_t *>(queries) + (uint64_t)qi * D_;
    for (uint32_t d = lane_id(); d < (uint32_t)kQueryWords; d += kWave) qlds[d] = d < D_ ? src[d] : 0u;
    qs = reinterpret_cast<const float *>(qlds);
  }

  // acc + (q_d - x_d)^2 for one element, each step rounded on its own
  __device__ __forceinline__ static float step(float acc, float qd, float xd) {
    const float t = __fsub_rn(qd, xd);
    return __fadd_rn(acc, __fmul_rn(t, t));
  }

  // Sequential distance of this lane's vector; ld4(i) returns bytes
  // [16i, 16i + 16) of the vector, ld1(d) the d-th float's bits.
  template <class Ld4, class Ld1>
  __device__ __forceinline__ float dist_lane(Ld4 ld4, Ld1 ld1) const {
    float acc = 0.0f;
    if constexpr (EXACT) {
      uint4 x[NV4];
#pragma unroll
      for (int i = 0; i < NV4; ++i) x[i] = ld4(i);
#pragma unroll
      for (int i = 0; i < NV4; ++i) {
        const float4 qv = *reinterpret_cast<const float4 *>(qs + 4 * i);
        acc = step(acc, qv.x, __uint_as_float(x[i].x));
        acc = step(acc, qv.y, __uint_as_float(x[i].y));
        acc = step(acc, qv.z, __uint_as_float(x[i].z));
        acc = step(acc, qv.w, __uint_as_float(x[i].w));
      }
    } else {
      for (uint32_t d0 = 0; d0 < D; d0 += kStep) {
        uint32_t x[kStep];
#pragma unroll
        for (int j = 0; j < kStep; ++j) x[j] = d0 + j < D ? ld1(d0 + j) : 0u;
#pragma unroll
        for (int j = 0; j < kStep; ++j)
          if (d0 + j < D) acc = step(acc, qs[d0 + j], __uint_as_float(x[j]));
      }
    }
    return acc;
  }

  __device__ __forceinline__ float dist_cached(__amdgpu_buffer_rsrc_t r, uint32_t off) const {
    return dist_lane([&](int i) { return coherent_load_u128(r, off + 16u * (uint32_t)i); },
                     [&](uint32_t d) { return coherent_load_u32(r, off + 4u * d); });
  }

  template <class OffOf>
  __device__ __forceinline__ uint64_t paged_keys(OffOf off_of, __amdgpu_buffer_rsrc_t crs, const uint32_t *cand,
                                                 uint32_t base, bool rdy, uint32_t slot, uint64_t) const {
    uint64_t key = kInfKey;
    if (rdy) {
      const uint32_t node = cand[base + lane_id()];
      const float d = dist_cached(crs, off_of(slot, node));
      key = ((uint64_t)__float_as_uint(d) << 32) | ((uint64_t)node << 1);
    }
    return key;
  }
};

// Resident kernel: rows of at most 32 J floats (J lines of 128 bytes), any
// arrangement and placement.  One lane sums a candidate's whole vector, but a
// lane that reads its own vector makes every 16-byte load instruction touch 64
// different lines; so the 8 lanes of a group read 8 vectors, one at a time,
// each lane 16 bytes of every 128, and the 16-byte blocks pass through LDS, 16
// vectors at a time, so that each lane gets the line of its own vector for the
// sequential sum (no VALU work moves them).  The lines of one batch of 64
// vectors are in flight at any time: as a line is taken out of its registers
// the same line of the next batch is read into them.  Bound by random line
// reads: 300k x 128, R=32, L=64, 5,000 queries 2.79 ms with a lane per vector
// (1.8 TB/s), 0.81 ms now (6.5 TB/s; such reads reach 6.8); 256-d 3.78 -> 1.27.
// EXACT: every line is whole (D = 32 J).
template <int J, bool EXACT = false>
struct MetricF32Lines {
  static constexpr int kQueryWords = 32 * J;
  static constexpr uint32_t kPadDist = 0x7F800000u;  // +inf
  // A line takes 32 registers: up to four lines, two waves per SIMD.  Long
  // frontiers meet more nodes than a 16 KB visited table records, and 32 KB
  // (the 32-bit table too) leave room for one.  Rows of one or two lines are
  // bound by filter, LDS and merge more than by the gather, and a second wave
  // covers these: it is worth more than the records, also where half of the
  // evaluations are repeats.  100k nodes, 5,000 queries, L=200, us a call with
  // 32 KB and one wave / 16 KB and two: 20 floats, R=16 1,292 / 867, R=64 W=8
  // 2,036 / 1,393 (repeats 1% / 21%); 64 floats 1,497 / 957, 2,647 / 1,977.
  // A batch that leaves one wave per SIMD anyway has the larger table and, for
  // three and four lines at any frontier, with it the room and the two batches
  // of a kernel for one wave (few_ht_log2; us a call with the full batch's
  // kernel / this one: 200k x 32, R=64, W=8, L=200, 1,024 queries 632 / 548;
  // 200k x 96, R=64, W=8, L=64, 700 queries 295 / 249, 90 floats 329 / 275).
  __host__ __device__ static constexpr int ht_log2(int kpl) { return J <= 2 || (J <= 4 && kpl == 1) ? 13 : 14; }
  __host__ __device__ static constexpr int few_ht_log2(int kpl) {
    return kpl > 1 || J == 3 || J == 4 ? 14 : ht_log2(kpl);
  }
  __host__ __device__ static constexpr int waves_per_simd(int, uint32_t table_words) {
    return J <= 4 && table_words <= 4096 ? 2 : 1;
  }
  __host__ __device__ static constexpr int grid_waves_per_simd(int kpl, uint32_t w) { return waves_per_simd(kpl, w); }
  // With one wave per SIMD nothing else covers the LDS passes and the sums, so
  // such a kernel is given room (`roomy`): 32 vectors per LDS pass, and the
  // compiler may overlap one line's sums with the next lines' passes and keep
  // the query in registers; for whole lines two batches are in flight (1M x
  // 96, L=128, W=8, 10k queries: 5.27 ms without any of it, 4.83 with the
  // ragged line's tests, 4.18 now; with the 32-bit table, 2^24 + 4,099 nodes,
  // R=16, 5,000 queries: L=64 906 us ragged and 838 whole, L=128 1,370 and
  // 1,288).  Not with four frontier registers: there they take the registers
  // the overlap needs (100k x 96, L=200, 5,000 queries: R=16 1,541 us with one
  // batch and 1,672 with two, R=64 2,650 and 2,883), nor with four lines,
  // whose second batch spills (100k x 128, R=16, L=100: 925 and 2,286).
  __host__ __device__ static constexpr bool roomy(int kpl, uint32_t w) { return waves_per_simd(kpl, w) == 1 && J <= 4; }
  __host__ __device__ static constexpr bool two_batches(int kpl, uint32_t w) {
    return EXACT && J <= 3 && roomy(kpl, w) && kpl <= 2;
  }
  __host__ __device__ static constexpr uint32_t stage_words(int kpl, uint32_t w) { return roomy(kpl, w) ? 1024 : 512; }
  static constexpr bool kLocators = false, kStream = false, kOffsets = false, kGathered = true;

  __device__ __forceinline__ static void pad_round(uint32_t *, uint64_t *, uint32_t, uint32_t, uint64_t) {}
  __device__ __forceinline__ static uint32_t cand_pos(uint32_t i) { return i; }
  __device__ __forceinline__ static uint32_t cand_word(const PageGeom &, uint32_t v) { return v; }

  // search_team: waves per query, and per SIMD at least
  __host__ __device__ static constexpr int team_waves(int kpl) { return kpl > 1 && J <= 4 ? 8 : 4; }
  __host__ __device__ static constexpr int team_per_simd() { return J <= 4 ? 2 : 1; }
  __host__ __device__ static constexpr int team_ht_log2(int kpl) { return kpl > 1 ? 14 : 13; }
  static constexpr int kTeamStageWords = 512;

  const float *qs;  // the query in LDS (wave-uniform reads), zeros past D
  uint4 *stage;     // LDS for sum_line, this wave's own: 1 KB per 8 vectors of a pass
  uint32_t D;

  __device__ __forceinline__ void set_stage(uint32_t *st) { stage = reinterpret_cast<uint4 *>(st); }

  // Copies the query into LDS; the caller synchronizes before use.
  __device__ __forceinline__ void load_query(const void *queries, uint32_t qi, uint32_t D_, uint32_t *qlds) {
    D = D_;
    const uint32_t *src = static_cast<const uint32_t *>(queries) + (uint64_t)qi * D_;
#pragma unroll
    for (uint32_t d0 = 0; d0 < (uint32_t)kQueryWords; d0 += kWave) {
      const uint32_t d = d0 + lane_id();
      if (d < (uint32_t)kQueryWords) qlds[d] = d < D_ ? src[d] : 0u;
    }
    qs = reinterpret_cast<const float *>(qlds);
  }

  // acc + (q_d - x_d)^2 for one element, each step rounded on its own
  __device__ __forceinline__ static float step(float acc, float qd, uint32_t xd) {
    const float t = __fsub_rn(qd, __uint_as_float(xd));
    return __fadd_rn(acc, __fmul_rn(t, t));
  }

  struct Line {
    uint32_t x[8][4];
  };
  struct Batch {
    Line line[J];
  };

  // Line j of the vectors of the group's 8 candidates: x[r][c] = float
  // 32 j + 4 gl + c of the vector of lane r * 8 + g (byte offset `off` in lane
  // r * 8 + g).  Blocks past the vector's last read the last one again; that
  // one may reach up to 12 bytes past the vector (the page array ends with
  // 16 spare bytes).
  __device__ __forceinline__ void load_line(const uint8_t *pages, uint64_t off, int j, Line &ln) const {
    const uint32_t l = lane_id(), g = l >> 3, gl = l & 7u;
    const uint32_t at = EXACT || j + 1 < J ? 32u * j + 4u * gl : min(32u * j + 4u * gl, (D - 1u) & ~3u);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint64_t o = __shfl(off, r * 8 + (int)g);
      const uint32_t *w = reinterpret_cast<const uint32_t *>(pages + o) + at;
      uint4 u;
      __builtin_memcpy(&u, __builtin_assume_aligned(w, 4), 16);
      ln.x[r][0] = u.x;
      ln.x[r][1] = u.y;
      ln.x[r][2] = u.z;
      ln.x[r][3] = u.w;
    }
  }

  // Block k of LDS row t sits at 16-byte position k ^ ((t >> 1) & 7): the
  // writes of one round cover 1 KB contiguously and the reads (lane t, row
  // t) spread 16 consecutive lanes over all 64 banks.
  __device__ __forceinline__ static uint32_t tpos(uint32_t row, uint32_t k) { return row * 8u + (k ^ ((row >> 1) & 7u)); }

  // acc over line j of this lane's vector: through LDS, lane i receives
  // y[k] = block k of its own vector's line (floats 32 j + 4 k .. + 3), so k
  // then the component visits d in increasing order.
  template <bool ROOMY>
  __device__ __forceinline__ float sum_line(float acc, const Line &ln, int j) const {
    constexpr uint32_t kRows = ROOMY ? 32 : 16;  // vectors per pass
    const uint32_t l = lane_id(), g = l >> 3, gl = l & 7u, t = l & (kRows - 1);
    uint4 y[8];
#pragma unroll
    for (uint32_t h = 0; h < kWave / kRows; ++h) {
#pragma unroll
      for (uint32_t rr = 0; rr < kRows / 8; ++rr) {
        const uint32_t r = h * (kRows / 8) + rr;
        stage[tpos(rr * 8u + g, gl)] = make_uint4(ln.x[r][0], ln.x[r][1], ln.x[r][2], ln.x[r][3]);
      }
      if (l / kRows == h) {
#pragma unroll
        for (int k = 0; k < 8; ++k) y[k] = stage[tpos(t, (uint32_t)k)];
      }
    }
    // the line's part of the query, read where it is used: taken out of the
    // loop over batches, the whole query would hold 32 registers per line
    int q0 = 32 * j;
    if constexpr (!ROOMY) asm volatile("" : "+s"(q0));
    if (EXACT || j + 1 < J) {
#pragma unroll
      for (int k = 0; k < 8; ++k) acc = step4(acc, q0 + 4 * k, y[k]);
    } else {
      // the vector's last line: rem floats; the query is 0 past them and so
      // is x made, which leaves the sum as it is
      const uint32_t rem = D - 32u * j;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (4u * k >= rem) break;
        if (4u * k + 4u > rem) {
          if (4u * k + 1u >= rem) y[k].y = 0u;
          if (4u * k + 2u >= rem) y[k].z = 0u;
          y[k].w = 0u;
        }
        acc = step4(acc, q0 + 4 * k, y[k]);
      }
    }
    // the line is summed here: sunk to where the distance is used, the sums
    // would keep every line's y until then
    if constexpr (!ROOMY) asm volatile("" : "+v"(acc));
    return acc;
  }
  __device__ __forceinline__ float step4(float acc, int d, const uint4 &x) const {
    const float4 qv = *reinterpret_cast<const float4 *>(qs + d);
    acc = step(acc, qv.x, x.x);
    acc = step(acc, qv.y, x.y);
    acc = step(acc, qv.z, x.z);
    return step(acc, qv.w, x.w);
  }

  __device__ __forceinline__ void issue(const uint8_t *pages, uint64_t off, Batch &b) const {
#pragma unroll
    for (int j = 0; j < J; ++j) load_line(pages, off, j, b.line[j]);
  }
  // Distance bits of the batch in b; the vectors at `next` take its place.
  template <bool ROOMY>
  __device__ __forceinline__ uint32_t dist_and_issue(const uint8_t *pages, uint64_t next, Batch &b) const {
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      acc = sum_line<ROOMY>(acc, b.line[j], j);
      if constexpr (!ROOMY) {
        load_line(pages, next, j, b.line[j]);
        __builtin_amdgcn_sched_barrier(0);  // no load moves ahead of the line it replaces
      }
    }
    if constexpr (ROOMY) issue(pages, next, b);
    return __float_as_uint(acc);
  }
  template <bool ROOMY>
  __device__ __forceinline__ uint32_t dist(const Batch &b) const {
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < J; ++j) acc = sum_line<ROOMY>(acc, b.line[j], j);
    return __float_as_uint(acc);
  }
  // Distance bits of one record (`off` the same in every lane).
  __device__ __forceinline__ uint32_t dist_one(const uint8_t *pages, uint64_t off) const {
    Batch b;
    issue(pages, off, b);
    return dist<false>(b);
  }
};

// Resident kernel: rows of at most 8 floats, at most two 16-byte blocks, which
// the lane that sums them reads itself.  A line gather would read such rows
// with eight lanes each and pass them through LDS: one load instruction per 8
// vectors and 10 LDS accesses per 16, where a lane's own block is one or two
// loads for all 64.  100k nodes, 5,000 queries, us a call with a lane per vector
// and dword loads / the line gather / here: 4 floats, R=64, W=8, L=64 420 / 435
// / 305; 8 floats 457 / 434 / 330; 4 floats, placed, R=32, L=200 941 / 1,834 /
// 744.  Rows of 9 to 16 floats (three or four blocks) are as fast either way.
struct MetricF32Own {
  static constexpr int kQueryWords = 8;
  static constexpr uint32_t kPadDist = 0x7F800000u;  // +inf
  // two waves and 16 KB, as MetricF32Lines of one line
  __host__ __device__ static constexpr int ht_log2(int) { return 13; }
  __host__ __device__ static constexpr int few_ht_log2(int kpl) { return kpl > 1 ? 14 : ht_log2(kpl); }
  __host__ __device__ static constexpr int waves_per_simd(int, uint32_t table_words) { return table_words > 4096 ? 1 : 2; }
  __host__ __device__ static constexpr int grid_waves_per_simd(int kpl, uint32_t w) { return waves_per_simd(kpl, w); }
  __host__ __device__ static constexpr bool roomy(int, uint32_t) { return false; }
  __host__ __device__ static constexpr bool two_batches(int, uint32_t) { return false; }
  __host__ __device__ static constexpr uint32_t stage_words(int, uint32_t) { return 512; }  // ids and slots only
  static constexpr bool kLocators = false, kStream = false, kOffsets = false, kGathered = true;
  __device__ __forceinline__ static void pad_round(uint32_t *, uint64_t *, uint32_t, uint32_t, uint64_t) {}
  __device__ __forceinline__ static uint32_t cand_pos(uint32_t i) { return i; }
  __device__ __forceinline__ static uint32_t cand_word(const PageGeom &, uint32_t v) { return v; }

  __host__ __device__ static constexpr int team_waves(int kpl) { return kpl > 1 ? 8 : 4; }
  __host__ __device__ static constexpr int team_per_simd() { return 2; }
  __host__ __device__ static constexpr int team_ht_log2(int kpl) { return kpl > 1 ? 14 : 13; }
  static constexpr int kTeamStageWords = 0;
  __device__ __forceinline__ void set_stage(uint32_t *) {}

  float q[8];  // zeros past D
  uint32_t D;

  __device__ __forceinline__ void load_query(const void *queries, uint32_t qi, uint32_t D_, uint32_t *) {
    D = D_;
    const float *src = static_cast<const float *>(queries) + (uint64_t)qi * D_;
#pragma unroll
    for (uint32_t d = 0; d < 8; ++d) q[d] = d < D_ ? src[d] : 0.0f;
  }

  struct Batch {
    uint4 x[2];
  };
  // The last block may reach up to 12 bytes past the vector: the page array
  // ends with 16 spare bytes.
  __device__ __forceinline__ void issue(const uint8_t *pages, uint64_t off, Batch &b) const {
    const uint32_t *w = reinterpret_cast<const uint32_t *>(pages + off);
    __builtin_memcpy(&b.x[0], __builtin_assume_aligned(w, 4), 16);
    b.x[1] = make_uint4(0u, 0u, 0u, 0u);
    if (D > 4) __builtin_memcpy(&b.x[1], __builtin_assume_aligned(w + 4, 4), 16);
  }
  // Both the query and, past D, the vector are made 0: adding (0 - 0)^2 leaves
  // the sum as it is.
  template <bool ROOMY>
  __device__ __forceinline__ uint32_t dist(const Batch &b) const {
    const uint32_t x[8] = {b.x[0].x, b.x[0].y, b.x[0].z, b.x[0].w, b.x[1].x, b.x[1].y, b.x[1].z, b.x[1].w};
    float acc = 0.0f;
#pragma unroll
    for (uint32_t d = 0; d < 8; ++d) {
      const float t = __fsub_rn(q[d], __uint_as_float(d < D ? x[d] : 0u));
      acc = __fadd_rn(acc, __fmul_rn(t, t));
    }
    return __float_as_uint(acc);
  }
  template <bool ROOMY>
  __device__ __forceinline__ uint32_t dist_and_issue(const uint8_t *pages, uint64_t next, Batch &b) const {
    const Batch now = b;
    issue(pages, next, b);
    return dist<ROOMY>(now);
  }
  __device__ __forceinline__ uint32_t dist_one(const uint8_t *pages, uint64_t off) const {
    Batch b;
    issue(pages, off, b);
    return dist<false>(b);
  }
};

}  // namespace gorio
