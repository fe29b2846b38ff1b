// HBM-resident beam search for small batches: a team of T wavefronts per
// query.
//
// The loop is search_resident's (search_resident.hpp) and so are its results;
// what differs is who does what.  With few queries the chip is idle and a
// query's time is a chain of round trips: lists, visited filter, vectors,
// merge.  One wave walks up to 256 candidates of an iteration in four chunks;
// here each wave takes 64 ids through the filter and 64 vectors through the
// distance, so an iteration is one trip for all lists and one for all vectors.
// Every wave keeps its own copy of the frontier and merges the same keys into
// it (those below the frontier's L-th key, gathered in LDS), so that no wave
// waits for another to choose the next beam.
//
// One iteration, with its four barriers:
//   select   every wave marks the beam in its own frontier;
//   expand   wave w reads ids 64 w .. 64 w + 63 of the beam group;
//   filter   look up | A | claim and write | B | read back, compact | C;
//   evaluate wave w's candidates, keys below the threshold into LDS | D;
//   merge    every wave, all of those keys.
// Bound by two dependent memory trips per iteration (lists, vectors; about 2.8
// us an iteration with the barriers and LDS steps between them).  1M x 128
// uint8, R=64, L=64, W=4: one query, the same again 100 -> 64 us a call, another
// each time 118 -> 78; 1,024 queries 197 -> 140; 200k x 96 float32, 32 queries
// 199 -> 124.  Touching the lists of all
// new candidates together with their vectors, so that the next beam's were in
// the caches, made both slower (82 and 142 us).
//
// The filter's steps are separated because a wave must not see another's claim
// of a bucket before that wave's ids are in it.
#pragma once

#include "search_resident.hpp"

namespace gorio {

template <int KPL, class M, class HT, int T>
__global__ __launch_bounds__(T *kWave, M::team_per_simd()) void search_team(ResidentParams p) {
  constexpr uint32_t kCap = T * kWave;  // ids per beam group
  constexpr bool kOffsets = !M::kLocators;

  __shared__ __align__(16) uint32_t ht[HT::kWords];
  __shared__ __align__(16) uint32_t cand[kCap];
  __shared__ __align__(16) uint64_t coff[kOffsets ? kCap : 1];
  __shared__ uint64_t keys[kCap];
  __shared__ uint32_t beam[KPL * kWave];
  __shared__ __align__(16) uint32_t qbuf[M::kQueryWords];
  __shared__ __align__(16) uint32_t stage[M::kTeamStageWords ? M::kTeamStageWords * T : 1];
  __shared__ uint32_t n_cand, n_lost, n_keys, next_qi;

  const uint32_t l = lane_id(), w = threadIdx.x / kWave;
  const uint32_t beams_per_group = min(kCap / p.R, (uint32_t)kWave);
  const uint32_t entry_word = M::cand_word(p.geom, p.entry);
  const uint64_t entry_off = vec_offset(p.geom, slot_of(p.geom, p.entry));

  unsigned long long n_eval = 0, n_reeval = 0, n_exp = 0, n_iter = 0;
  if (threadIdx.x == 0) n_cand = n_lost = n_keys = 0;

  for (uint32_t qi = blockIdx.x; qi < p.nq;) {
    HT::template clear<T>(ht);
    M m;
    m.load_query(p.queries, qi, p.D, qbuf);
    m.set_stage(stage + M::kTeamStageWords * w);
    __syncthreads();

    bool forgot = false;  // some node may have been evaluated twice
    uint64_t F[KPL];
#pragma unroll
    for (int r = 0; r < KPL; ++r) F[r] = kInfKey;
    {
      const uint32_t d = m.dist_one(p.pages, entry_off);
      if (l == 0) F[0] = ((uint64_t)d << 32) | ((uint64_t)p.entry << 1);
      if (threadIdx.x == 0) {
        bool rec;
        HT::test_and_set(ht, p.entry, true, rec);
      }
      ++n_eval;
    }
    __syncthreads();

    for (uint32_t guard = 0; guard <= p.n; ++guard) {
      // ---- select (every wave writes the same beam) -------------------------
      uint32_t nbeam = 0;
#pragma unroll
      for (int r = 0; r < KPL; ++r) {
        const uint32_t e = r * kWave + l;
        bool unexp = e < p.L && F[r] != kInfKey && !(F[r] & 1ull);
        uint64_t mk = ballot(unexp);
        uint32_t rank = nbeam + lanes_below(mk);
        if (unexp && rank < p.W) {
          beam[rank] = key_id(F[r]);
          F[r] |= 1ull;
        }
        nbeam += (uint32_t)__popcll(mk);
      }
      if (nbeam > p.W) nbeam = p.W;
      if (nbeam == 0) break;
      asm volatile("" ::: "memory");  // LDS operations of one wave are in order
      n_exp += nbeam;
      ++n_iter;

      for (uint32_t b0 = 0; b0 < nbeam; b0 += beams_per_group) {
        // ---- expand: this lane's id and its list's degree, one trip ----------
        const uint32_t nslots = min(nbeam - b0, beams_per_group) * p.R;
        const uint32_t my = w * kWave + l;
        const uint32_t pos = min(my, nslots - 1);
        const uint32_t b = fastdiv(pos, p.Rdiv), j = pos - b * p.R;
        const uint8_t *adj = p.pages + adj_offset(p.geom, slot_of(p.geom, beam[b0 + b]));
        const uint32_t deg = min(*reinterpret_cast<const uint32_t *>(adj), p.R);
        const uint32_t id[1] = {reinterpret_cast<const uint32_t *>(adj + 4)[j]};
        const bool valid[1] = {my < nslots && j < deg && id[0] < p.n};
        [[maybe_unused]] uint32_t slot = 0;
        if constexpr (kOffsets) slot = slot_of(p.geom, valid[0] ? id[0] : p.entry);
        // ---- filter -----------------------------------------------------------
        typename HT::template Probe<1> pr;
        HT::look(ht, id, valid, true, pr);
        __syncthreads();  // A
        if (threadIdx.x == 0) n_keys = 0;
        HT::claim(ht, pr);
        __syncthreads();  // B
        bool isnew[1], recorded[1];
        HT::settle(ht, pr, isnew, recorded);
        const uint64_t mnew = ballot(isnew[0]);
        if (mnew != 0) {
          const uint64_t mlost = ballot(isnew[0] && !recorded[0]);
          uint32_t base = 0;
          if (l == 0) {
            base = atomicAdd(&n_cand, (uint32_t)__popcll(mnew));
            if (mlost) atomicAdd(&n_lost, (uint32_t)__popcll(mlost));
          }
          base = first_lane_value(base);
          if (isnew[0]) {
            const uint32_t at = M::cand_pos(base + lanes_below(mnew));
            cand[at] = M::cand_word(p.geom, id[0]);
            if constexpr (kOffsets) coff[at] = vec_offset(p.geom, slot);
          }
        }
        __syncthreads();  // C
        const uint32_t cnt = n_cand, lost = n_lost;
        n_eval += cnt;
        n_reeval += lost;
        forgot |= lost != 0;

        // ---- evaluate -----------------------------------------------------------
        const uint32_t c0 = w * kWave;
        if (c0 < cnt) {
          // the rest of the last chunk reads the entry's vector
          if (c0 + l >= cnt) {
            cand[M::cand_pos(c0 + l)] = entry_word;
            if constexpr (kOffsets) coff[c0 + l] = entry_off;
          }
          asm volatile("" ::: "memory");
          uint64_t key;
          if constexpr (M::kStream) {
            typename M::Chunk ck;
            m.chunk_issue(p.pages, p.geom, cand, coff, c0, ck);
            key = m.chunk_key(p.geom, cand, c0, cnt, ck);
          } else {
            static_assert(M::kGathered, "a streaming or a line-gathering policy");
            typename M::Batch bt;
            m.issue(p.pages, coff[c0 + l], bt);
            key = ((uint64_t)m.template dist<false>(bt) << 32) | ((uint64_t)cand[c0 + l] << 1);
            if (c0 + l >= cnt) key = kInfKey;
          }
          const bool pass = key < frontier_at<KPL>(F, p.L - 1);
          const uint64_t mp = ballot(pass);
          if (mp != 0) {
            uint32_t base = 0;
            if (l == 0) base = atomicAdd(&n_keys, (uint32_t)__popcll(mp));
            base = first_lane_value(base);
            if (pass) keys[base + lanes_below(mp)] = key;
          }
        }
        __syncthreads();  // D
        if (threadIdx.x == 0) n_cand = n_lost = 0;

        // ---- merge ----------------------------------------------------------------
        const uint32_t nk = n_keys;
        for (uint32_t k0 = 0; k0 < nk; k0 += kWave)
          merge_keys<KPL, false>(F, k0 + l < nk ? keys[k0 + l] : kInfKey, forgot, p.L);
      }
    }

    // ---- result: first k slots of F -------------------------------------------
    if (w == 0) {
#pragma unroll
      for (int r = 0; r < KPL; ++r) {
        const uint32_t e = r * kWave + l;
        if (e < p.k) {
          const bool ok = F[r] != kInfKey;
          p.out_ids[(uint64_t)qi * p.k + e] = ok ? key_id(F[r]) : kNoEdge;
          p.out_dists[(uint64_t)qi * p.k + e] = ok ? (uint32_t)(F[r] >> 32) : M::kPadDist;
        }
      }
    }
    if (threadIdx.x == 0) next_qi = gridDim.x + (uint32_t)(atomicAdd(p.next_query, 1ull) - p.next_base);
    __syncthreads();
    qi = next_qi;
    __syncthreads();
  }

  if (threadIdx.x == 0) {
    atomicAdd(&p.stats[0], n_eval);
    atomicAdd(&p.stats[1], n_reeval);
    atomicAdd(&p.stats[2], n_exp);
    atomicAdd(&p.stats[3], n_iter);
  }
}

}  // namespace gorio
