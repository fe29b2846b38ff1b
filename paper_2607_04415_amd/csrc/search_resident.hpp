// HBM-resident beam search: one wavefront per query.
//
// Per query the wave keeps the frontier F (the L best keys of the evaluated
// set, ascending) in registers, 64 * KPL slots, slot e = r * 64 + lane, and its
// visited filter in LDS.  Key = (distance bits << 32) | (node id << 1) |
// expanded bit: ties order by id, and the flag rides along through the
// sorting networks.  One iteration (GORIO Sec. 1 / Sec. 2.2: expand nodes,
// compute distances, update the frontier):
//   select  - the first W unexpanded slots of F (ballot + prefix count);
//   expand  - one round trip reads the degree and id list of every chosen
//             node of a beam group (up to 256 ids, 4 per lane); with float32
//             line-gathered rows (no placement) a beam of several groups reads
//             the next group's lists while the current one is filtered and
//             evaluated;
//   filter  - ids already in the visited filter are dropped (LDS atomics),
//             the rest compacted into an LDS candidate list;
//   evaluate- one round trip gathers a batch of candidate vectors by whole
//             lines, 8 lanes per vector; the distance policy (metric.hpp)
//             turns them into keys: uint8 with v_dot4_u32_u8, float32 with one
//             lane per vector (the blocks reach it through LDS) and the
//             sequential rounded sum;
//   merge   - only keys below F's L-th key can enter: a few are inserted by
//             rank (ballot + DPP shift), many are bitonic-sorted per 64-lane
//             chunk and bitonic-merged into F.
#pragma once

#include "metric.hpp"

namespace gorio {

struct ResidentParams {
  const uint8_t *pages;    // num_pages * page_bytes, HBM
  PageGeom geom;
  uint32_t n;
  uint32_t D;              // vector elements (uint8: a multiple of 4)
  uint32_t R;              // id slots per record
  FastDiv Rdiv;            // division by R
  uint32_t entry;
  const void *queries;     // nq x D elements
  uint32_t nq;
  uint32_t k, L, W;
  uint32_t *out_ids;       // nq x k
  uint32_t *out_dists;     // nq x k distance bits (int32 or float32)
  unsigned long long *stats;  // [evaluations, reevaluations, expansions, iterations]
  // Queries past the first grid are handed out by a counter that only grows:
  // every completed query takes one ticket, so a launch adds exactly nq, and
  // next_base is the counter's value when this launch starts (no reset between
  // launches).
  unsigned long long *next_query;
  unsigned long long next_base;
};

// Evaluates NCH chunks of 64 compacted candidates (streaming metrics) and
// merges their keys into F, with two chunks in flight.
template <int NCH, int KPL, class M>
__device__ __forceinline__ void eval_chunks(const M &m, const ResidentParams &p, const uint32_t *cand,
                                            const uint64_t *coff, uint32_t cnt, uint64_t (&F)[KPL], bool forgot) {
  typename M::Chunk A, B;
  m.chunk_issue(p.pages, p.geom, cand, coff, 0, A);
  if constexpr (NCH > 1) m.chunk_issue(p.pages, p.geom, cand, coff, kWave, B);
  uint64_t key = m.chunk_key(p.geom, cand, 0, cnt, A);
  if constexpr (NCH > 2) m.chunk_issue(p.pages, p.geom, cand, coff, 2 * kWave, A);
  merge_keys<KPL>(F, key, forgot, p.L);
  if constexpr (NCH > 1) {
    key = m.chunk_key(p.geom, cand, kWave, cnt, B);
    if constexpr (NCH > 3) m.chunk_issue(p.pages, p.geom, cand, coff, 3 * kWave, B);
    merge_keys<KPL>(F, key, forgot, p.L);
  }
  if constexpr (NCH > 2) merge_keys<KPL>(F, m.chunk_key(p.geom, cand, 2 * kWave, cnt, A), forgot, p.L);
  if constexpr (NCH > 3) merge_keys<KPL>(F, m.chunk_key(p.geom, cand, 3 * kWave, cnt, B), forgot, p.L);
}

// A group's cnt compacted candidates, 64 at a time, as the float32 line gather
// takes them: lane l's candidate of the batch t ahead (past the count: any
// record, its key is dropped).
//
// In LDS, in words of their own.
template <bool N2S>
struct LdsCandidates {
  const uint32_t *cand;
  const uint64_t *off;  // byte offsets, with a placement
  uint32_t cnt, entry;
  uint64_t entry_off;
  uint32_t first = 0;

  __device__ __forceinline__ uint32_t id(int t) const { return cand[first + t * kWave + lane_id()]; }
  __device__ __forceinline__ uint64_t offset(const PageGeom &geom, int t) const {
    const uint32_t i = first + t * kWave + lane_id();
    if constexpr (N2S) return i < cnt ? off[i] : entry_off;
    else return vec_offset(geom, i < cnt ? cand[i] : entry);
  }
  __device__ __forceinline__ void next() { first += kWave; }
};
// In registers: their words in LDS are then the stage's, which the lines pass
// through.
template <bool N2S>
struct LaneCandidates {
  uint32_t ids[kCandCap / kWave];
  uint32_t slot[N2S ? kCandCap / kWave : 1];  // identity placement: slot = id

  __device__ __forceinline__ void read(const uint32_t *cand, const uint32_t *slots, uint32_t cnt, uint32_t entry,
                                       uint32_t entry_slot) {
#pragma unroll
    for (int t = 0; t < kCandCap / kWave; ++t) {
      if (t * kWave >= cnt) break;
      const uint32_t i = t * kWave + lane_id();
      ids[t] = i < cnt ? cand[i] : entry;
      if constexpr (N2S) slot[t] = i < cnt ? slots[i] : entry_slot;
    }
  }
  __device__ __forceinline__ uint32_t id(int t) const { return ids[t]; }
  __device__ __forceinline__ uint64_t offset(const PageGeom &geom, int t) const {
    if constexpr (N2S) return vec_offset(geom, slot[t]);
    else return vec_offset(geom, ids[t]);
  }
  __device__ __forceinline__ void next() {
#pragma unroll
    for (int t = 0; t + 1 < kCandCap / kWave; ++t) {
      ids[t] = ids[t + 1];
      if constexpr (N2S) slot[t] = slot[t + 1];
    }
  }
};

// Evaluates cnt > 0 candidates with the float32 line gather, 64 at a time, and
// merges their keys into F.  The last batch has its own copy so that every
// batch before it issues the same loads and the waits stay exact.
template <int KPL, class M, bool ROOMY, class Cands>
__device__ __forceinline__ void eval_lines(const M &m, const ResidentParams &p, Cands &c, uint32_t cnt,
                                           uint64_t (&F)[KPL], bool forgot) {
  const uint32_t l = lane_id();
  typename M::Batch b;
  m.issue(p.pages, c.offset(p.geom, 0), b);
  uint32_t c0 = 0;
  for (; c0 + kWave < cnt; c0 += kWave) {
    const uint32_t d = m.template dist_and_issue<ROOMY>(p.pages, c.offset(p.geom, 1), b);
    merge_keys<KPL, false>(F, ((uint64_t)d << 32) | ((uint64_t)c.id(0) << 1), forgot, p.L);
    c.next();
  }
  const uint32_t d = m.template dist<ROOMY>(b);
  const uint64_t key = ((uint64_t)d << 32) | ((uint64_t)c.id(0) << 1);
  merge_keys<KPL, false>(F, c0 + l < cnt ? key : kInfKey, forgot, p.L);
}

// The same with two batches in flight (policies with one wave per SIMD, whose
// gathers nothing else would overlap): NCH batches, a fixed schedule each.
template <int NCH, int KPL, class M, bool ROOMY, class Cands>
__device__ __forceinline__ void eval_lines2(const M &m, const ResidentParams &p, const Cands &c, uint32_t cnt,
                                            uint64_t (&F)[KPL], bool forgot) {
  const uint32_t l = lane_id();
  typename M::Batch A, B;
  auto merge = [&](int t, uint32_t d) {
    const uint64_t key = ((uint64_t)d << 32) | ((uint64_t)c.id(t) << 1);
    merge_keys<KPL, false>(F, t * kWave + l < cnt ? key : kInfKey, forgot, p.L);
  };
  m.issue(p.pages, c.offset(p.geom, 0), A);
  if constexpr (NCH > 1) m.issue(p.pages, c.offset(p.geom, 1), B);
  if constexpr (NCH > 2) merge(0, m.template dist_and_issue<ROOMY>(p.pages, c.offset(p.geom, 2), A));
  else merge(0, m.template dist<ROOMY>(A));
  if constexpr (NCH > 3) merge(1, m.template dist_and_issue<ROOMY>(p.pages, c.offset(p.geom, 3), B));
  else if constexpr (NCH > 1) merge(1, m.template dist<ROOMY>(B));
  if constexpr (NCH > 2) merge(2, m.template dist<ROOMY>(A));
  if constexpr (NCH > 3) merge(3, m.template dist<ROOMY>(B));
}

template <int KPL, class M, bool TWO, bool ROOMY, class Cands>
__device__ __forceinline__ void eval_group(const M &m, const ResidentParams &p, Cands &c, uint32_t cnt,
                                           uint64_t (&F)[KPL], bool forgot) {
  if constexpr (TWO) {
    switch ((cnt + kWave - 1) / kWave) {
      case 1: eval_lines2<1, KPL, M, ROOMY>(m, p, c, cnt, F, forgot); break;
      case 2: eval_lines2<2, KPL, M, ROOMY>(m, p, c, cnt, F, forgot); break;
      case 3: eval_lines2<3, KPL, M, ROOMY>(m, p, c, cnt, F, forgot); break;
      case 4: eval_lines2<4, KPL, M, ROOMY>(m, p, c, cnt, F, forgot); break;
      default: break;
    }
  } else if (cnt != 0) {
    eval_lines<KPL, M, ROOMY>(m, p, c, cnt, F, forgot);
  }
}

// LDS of a search_resident workgroup.  launch_bounds cannot see it, so the sum
// is held against the share of the waves that are meant to run: 160 KB over
// four SIMDs.  The compacted candidates (ids, with a placement also byte
// offsets) have words of their own; where that would cost a wave, the line
// gather keeps ids and slots in the stage's words and takes them into
// registers before the first line passes through (100k x 96, placed, 5,000
// queries, L=200: 2,741 us with three workgroups per CU of 41 KB, 2,043 with
// four; L=64, seven workgroups of 22 KB and eight: 1,097 and 1,062).  Where
// they fit, their own words are the faster form (up to 2%).
template <int KPL, class M, class HT, bool N2S>
struct ResidentLds {
  static constexpr int kCompiled = M::waves_per_simd(KPL, HT::kWords), kGrid = M::grid_waves_per_simd(KPL, HT::kWords);
  static constexpr uint32_t kShare = 160 * 1024 / 4 / (kCompiled < kGrid ? kCompiled : kGrid);
  static constexpr uint32_t kStageWords = M::stage_words(KPL, HT::kWords);
  static constexpr bool kPlaced = M::kOffsets || (M::kGathered && N2S);
  static constexpr uint32_t kOwnBytes = 4 * (kCandCap + (kPlaced ? 2 * kCandCap : 0));
  // (a query kept in registers leaves its one word unused)
  static constexpr uint32_t kOtherBytes =
      4 * (HT::kWords + KPL * kWave + (M::kQueryWords > 1 ? M::kQueryWords : 0) + kStageWords);
  static constexpr bool kInStage = M::kGathered && kOtherBytes + kOwnBytes > kShare;
  static_assert(!kInStage || kStageWords >= 2 * kCandCap, "ids and slots fit the stage");
  static constexpr bool kOffsets = kPlaced && !kInStage, kSlots = kPlaced && kInStage;
  static constexpr uint32_t kBytes = kOtherBytes + (kInStage ? 0 : kOwnBytes);
  static constexpr bool kFits = kBytes <= kShare;
  // The compiler schedules for no more waves than the LDS it sees leaves room
  // for; a kernel that is to be scheduled for more than run takes its table as
  // the launch's LDS (16-bit tables).
  static constexpr bool kHidden = kBytes > 160 * 1024 / 4 / kCompiled && HT::kWords <= 4096;
  static constexpr uint32_t kLaunchBytes = kHidden ? 4 * HT::kWords : 0;
};

// Waves per SIMD and the visited table from the distance policy
// (M::waves_per_simd, M::ht_log2): one wave's gathers overlap the others'
// filtering and merging.  The grid is as large as the chip holds at
// once; workgroup b starts with query b and then takes the next unclaimed
// query from a global counter, so the XCDs and CUs that finish early take
// more queries and the batch ends when the last queries end, wherever they
// run.
template <int KPL, class M, class HT, bool N2S>
__global__ __launch_bounds__(kWave, M::waves_per_simd(KPL, HT::kWords)) void search_resident(ResidentParams p) {
  constexpr int kIdsPerLane = kCandCap / kWave;
  using Lds = ResidentLds<KPL, M, HT, N2S>;
  static_assert(Lds::kFits, "the waves this kernel is compiled for fit a CU's LDS");

  extern __shared__ __align__(16) uint32_t launch_lds[];
  __shared__ __align__(16) uint32_t static_table[Lds::kLaunchBytes ? 1 : HT::kWords];
  uint32_t *const ht = Lds::kLaunchBytes ? launch_lds : static_table;
  __shared__ __align__(16) uint32_t own_cand[Lds::kInStage ? 1 : kCandCap];
  __shared__ uint32_t beam[KPL * kWave];  // W <= L
  // candidates' byte offsets (or slots), worked out as they are compacted: the
  // placement is then looked up beside the filter, for all ids of a group at once
  constexpr bool kOffsets = Lds::kOffsets, kSlots = Lds::kSlots;
  __shared__ __align__(16) uint64_t coff[kOffsets ? kCandCap : 1];
  __shared__ __align__(16) uint32_t qbuf[M::kQueryWords];
  __shared__ __align__(16) uint32_t stage[Lds::kStageWords ? Lds::kStageWords : 1];
  uint32_t *const cand = Lds::kInStage ? stage : own_cand;
  [[maybe_unused]] uint32_t *const cand_slot = stage + kCandCap;

  const int l = lane_id();
  const uint32_t beams_per_group = min(kCandCap / p.R, (uint32_t)kWave);
  const uint32_t entry_word = M::cand_word(p.geom, p.entry);
  const uint32_t entry_slot = slot_ct<N2S>(p.geom, p.entry);
  const uint64_t entry_off = vec_offset(p.geom, entry_slot);

  unsigned long long n_eval = 0, n_reeval = 0, n_exp = 0, n_iter = 0;

  for (uint32_t qi = blockIdx.x; qi < p.nq;) {
    HT::clear(ht);
    M m;
    m.load_query(p.queries, qi, p.D, qbuf);
    m.set_stage(stage);
    __syncthreads();

    uint32_t ht_used = 0;
    bool forgot = false;  // some node may have been evaluated twice

    // V = {entry}
    uint64_t F[KPL];
#pragma unroll
    for (int r = 0; r < KPL; ++r) F[r] = kInfKey;
    {
      const uint32_t d = m.dist_one(p.pages, entry_off);
      if (l == 0) {
        F[0] = ((uint64_t)d << 32) | ((uint64_t)p.entry << 1);
        bool rec;
        HT::test_and_set(ht, p.entry, true, rec);
      }
      ht_used = 1;
      ++n_eval;
    }
    __syncthreads();

    for (uint32_t guard = 0; guard <= p.n; ++guard) {
      // ---- select: first W unexpanded slots of F, in order -----------------
      uint32_t nbeam = 0;
#pragma unroll
      for (int r = 0; r < KPL; ++r) {
        const uint32_t e = r * kWave + l;
        bool unexp = e < p.L && F[r] != kInfKey && !(F[r] & 1ull);
        uint64_t m = ballot(unexp);
        uint32_t rank = nbeam + lanes_below(m);
        if (unexp && rank < p.W) {
          beam[rank] = key_id(F[r]);
          F[r] |= 1ull;
        }
        nbeam += (uint32_t)__popcll(m);
      }
      if (nbeam > p.W) nbeam = p.W;
      if (nbeam == 0) break;
      __syncthreads();
      n_exp += nbeam;
      ++n_iter;

      // ---- expand: degrees (lane b) and all id slots of a beam group at once.
      // Loads are unconditional (lanes past the group read the group's first
      // record) so that no branch separates them: one round trip per group.
      // Float32 line-gathered rows (W=8, R=64: two groups per beam) read the
      // next group's lists while this group is filtered and evaluated, so only
      // the first group's round trip is exposed.  Other metrics read a group's
      // lists when they reach it: a uint8 beam at W=4 fits one group, and a
      // second set of list registers would only constrain the allocator.  So do
      // rows with a placement, whose slot lookups between lists and gather wait
      // for every load before them, the next group's lists too; for the same
      // reason they keep one batch in flight (96 floats, placed, 5,000 queries,
      // L=128, W=8, us a call with both / without: 6k nodes, R=32 864 / 773; 600k
      // nodes 1,393 / 1,302).
      constexpr bool kAhead = M::kGathered && !N2S;
      struct AdjLoad {
        uint64_t off;  // lane b: adjacency block of the group's beam b
        uint32_t deg;  // lane b: its degree
        uint32_t ids[kIdsPerLane];
      };
      auto issue_adj = [&](uint32_t b0, AdjLoad &A) {
        const uint32_t nb = min(nbeam - b0, beams_per_group);
        const uint32_t nslots = nb * p.R;
        const uint32_t my_beam = beam[b0 + min((uint32_t)l, nb - 1)];
        A.off = adj_offset(p.geom, slot_ct<N2S>(p.geom, my_beam));
        A.deg = *reinterpret_cast<const uint32_t *>(p.pages + A.off);
#pragma unroll
        for (int t = 0; t < kIdsPerLane; ++t) {
          const uint32_t pos = min(t * kWave + (uint32_t)l, nslots - 1);
          const uint32_t b = fastdiv(pos, p.Rdiv);
          const uint64_t adj = __shfl(A.off, (int)b);
          A.ids[t] = reinterpret_cast<const uint32_t *>(p.pages + adj + 4)[pos - b * p.R];
        }
      };
      [[maybe_unused]] AdjLoad cur, nxt;
      if constexpr (kAhead) issue_adj(0, cur);
      for (uint32_t b0 = 0; b0 < nbeam; b0 += beams_per_group) {
        const uint32_t nb = min(nbeam - b0, beams_per_group);
        const uint32_t nslots = nb * p.R;
        uint32_t ids[kIdsPerLane];
        bool valid[kIdsPerLane];
        if constexpr (kAhead) {
          if (b0 + beams_per_group < nbeam) issue_adj(b0 + beams_per_group, nxt);
#pragma unroll
          for (int t = 0; t < kIdsPerLane; ++t) {
            const uint32_t pos = min(t * kWave + (uint32_t)l, nslots - 1);
            const uint32_t b = fastdiv(pos, p.Rdiv);
            const uint32_t deg = min((uint32_t)__shfl((int)cur.deg, (int)b), p.R);
            ids[t] = cur.ids[t];
            valid[t] = (uint32_t)(t * kWave + l) < nslots && pos - b * p.R < deg && ids[t] < p.n;
          }
        } else {
          const uint32_t my_beam = beam[b0 + min((uint32_t)l, nb - 1)];
          const uint64_t my_adj = adj_offset(p.geom, slot_ct<N2S>(p.geom, my_beam));
          const uint32_t my_deg = *reinterpret_cast<const uint32_t *>(p.pages + my_adj);
          uint32_t slot_beam[kIdsPerLane], slot_j[kIdsPerLane];
#pragma unroll
          for (int t = 0; t < kIdsPerLane; ++t) {
            const uint32_t pos = min(t * kWave + (uint32_t)l, nslots - 1);
            const uint32_t b = fastdiv(pos, p.Rdiv);
            slot_beam[t] = b;
            slot_j[t] = pos - b * p.R;
          }
#pragma unroll
          for (int t = 0; t < kIdsPerLane; ++t) {
            const uint64_t adj = __shfl(my_adj, (int)slot_beam[t]);
            ids[t] = reinterpret_cast<const uint32_t *>(p.pages + adj + 4)[slot_j[t]];
          }
#pragma unroll
          for (int t = 0; t < kIdsPerLane; ++t) {
            const uint32_t deg = min((uint32_t)__shfl((int)my_deg, (int)slot_beam[t]), p.R);
            valid[t] = (uint32_t)(t * kWave + l) < nslots && slot_j[t] < deg && ids[t] < p.n;
          }
        }
        [[maybe_unused]] uint32_t slot[kIdsPerLane];
        if constexpr (kOffsets || kSlots) {
#pragma unroll
          for (int t = 0; t < kIdsPerLane; ++t) slot[t] = slot_ct<N2S>(p.geom, valid[t] ? ids[t] : p.entry);
        }
        // ---- filter through the visited table, compact the new ids ------------
        bool isnew[kIdsPerLane], recorded[kIdsPerLane];
        HT::template test_and_set_n<kIdsPerLane>(ht, ids, valid, ht_used < HT::kLimit, isnew, recorded);
        uint32_t cnt = 0;
#pragma unroll
        for (int t = 0; t < kIdsPerLane; ++t) {
          const uint64_t mnew = ballot(isnew[t]);
          const uint64_t mrec = ballot(recorded[t]);
          if (isnew[t]) {
            const uint32_t at = M::cand_pos(cnt + lanes_below(mnew));
            cand[at] = M::cand_word(p.geom, ids[t]);
            if constexpr (kOffsets) coff[at] = vec_offset(p.geom, slot[t]);
            if constexpr (kSlots) cand_slot[at] = slot[t];
          }
          cnt += (uint32_t)__popcll(mnew);
          ht_used += (uint32_t)__popcll(mrec);
          const uint32_t lost = (uint32_t)__popcll(mnew & ~mrec);
          n_reeval += lost;
          forgot |= lost != 0;
        }
        M::pad_round(cand, coff, cnt, entry_word, entry_off);
        __syncthreads();
        n_eval += cnt;

        // ---- evaluate and merge -----------------------------------------------
        if constexpr (M::kStream) {
          // chunks of 64 vectors, two in flight: the next chunk's gathers are
          // outstanding while this one is reduced and merged (a fixed schedule
          // per chunk count keeps every wait exact)
          static_assert(kCandCap == 4 * kWave, "at most four chunks");
          switch ((cnt + kWave - 1) / kWave) {
            case 1: eval_chunks<1, KPL>(m, p, cand, coff, cnt, F, forgot); break;
            case 2: eval_chunks<2, KPL>(m, p, cand, coff, cnt, F, forgot); break;
            case 3: eval_chunks<3, KPL>(m, p, cand, coff, cnt, F, forgot); break;
            case 4: eval_chunks<4, KPL>(m, p, cand, coff, cnt, F, forgot); break;
            default: break;
          }
        } else if constexpr (M::kGathered) {
          constexpr bool kTwo = !N2S && M::two_batches(KPL, HT::kWords), kRoomy = M::roomy(KPL, HT::kWords);
          if constexpr (Lds::kInStage) {
            LaneCandidates<N2S> c;
            c.read(cand, cand_slot, cnt, p.entry, entry_slot);
            asm volatile("" ::: "memory");  // read before the stage is written (LDS operations of one wave are in order)
            eval_group<KPL, M, kTwo, kRoomy>(m, p, c, cnt, F, forgot);
          } else {
            LdsCandidates<N2S> c{cand, coff, cnt, p.entry, entry_off};
            eval_group<KPL, M, kTwo, kRoomy>(m, p, c, cnt, F, forgot);
          }
        } else {
          // batches of kBatch vectors, one round trip each
          for (uint32_t c0 = 0; c0 < cnt; c0 += M::kBatch) {
            uint64_t key[M::kChunks];
            m.template resident_keys<N2S>(p.pages, p.geom, cand, c0, cnt, p.entry, key);
#pragma unroll
            for (int c = 0; c < M::kChunks; ++c) merge_keys<KPL, KPL == 1>(F, key[c], forgot, p.L);
          }
        }
        __syncthreads();
        if constexpr (kAhead) cur = nxt;
      }
    }

    // ---- result: first k slots of F -------------------------------------------
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
      const uint32_t e = r * kWave + l;
      if (e < p.k) {
        const bool ok = F[r] != kInfKey;
        p.out_ids[(uint64_t)qi * p.k + e] = ok ? key_id(F[r]) : kNoEdge;
        p.out_dists[(uint64_t)qi * p.k + e] = ok ? (uint32_t)(F[r] >> 32) : M::kPadDist;
      }
    }
    uint32_t next = 0;
    if (l == 0) next = (uint32_t)(atomicAdd(p.next_query, 1ull) - p.next_base);
    qi = gridDim.x + first_lane_value(next);
  }

  if (l == 0) {
    atomicAdd(&p.stats[0], n_eval);
    atomicAdd(&p.stats[1], n_reeval);
    atomicAdd(&p.stats[2], n_exp);
    atomicAdd(&p.stats[3], n_iter);
  }
}

}  // namespace gorio
