// Kernel launchers.  Each dtype's kernel variants are instantiated in a
// translation unit of their own (resident_u8.hip, resident_f32.hip,
// paged_u8.hip, paged_f32.hip) so that they compile in parallel.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "search_paged.hpp"
#include "search_resident.hpp"
#include "search_team.hpp"

namespace gorio {

// Resident search: one wave per query at a time, at most `grid` workgroups
// (queries past the grid are handed out by the kernel's counter).
hipError_t launch_resident_u8(const ResidentParams &p, int grid, hipStream_t s);
hipError_t launch_resident_f32(const ResidentParams &p, int grid, hipStream_t s);

// Paged search: the persistent kernel (fill waves + query waves).  With
// grid == pp.fill_waves it runs only the fill waves.
hipError_t launch_paged_u8(const PagedParams &pp, int grid, hipStream_t s);
hipError_t launch_paged_f32(const PagedParams &pp, int grid, hipStream_t s);

// Host-scheduled lanes: one workgroup per listed lane, or (no list) the
// persistent launch of fill waves, the run ring's tail mirror and executors.
hipError_t launch_rounds_u8(const PagedParams &pp, const RoundParams &rp, int grid, hipStream_t s);
hipError_t launch_rounds_f32(const PagedParams &pp, const RoundParams &rp, int grid, hipStream_t s);

// 32-bit words of one lane's saved state for a search with frontier size L.
inline uint32_t lane_state_words(uint32_t L) {
  const size_t b = L <= 64 ? sizeof(QSlot<1>) : L <= 128 ? sizeof(QSlot<2>) : sizeof(QSlot<4>);
  return (uint32_t)((b + 3) / 4);
}

// Visited tables of the resident kernel: 16-bit entries (2^M::ht_log2 of
// them) when every id fits that table's domain, else 8192 32-bit entries.
using ResidentHtLarge = VisitedLds<13>;

namespace detail {

// Workgroups of a resident kernel's grid: one per wave slot the device holds
// at once, but at most `grid_waves_per_simd` per SIMD (queries beyond the grid
// are taken from the kernel's counter).
template <auto Kernel, int grid_waves_per_simd, uint32_t lds>
hipError_t resident_slots(int &slots) {
  static int held = 0;  // per kernel
  if (held == 0) {
    constexpr int kSimdsPerCu = 4;
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(Kernel), kWave, lds);
    if (e != hipSuccess) return e;
    held = std::max(1, cus * std::min(per_cu, kSimdsPerCu * grid_waves_per_simd));
  }
  slots = held;
  return hipSuccess;
}

// `most`: do nothing (done = false) with more queries than the grid's workgroups.
template <int KPL, class M, class HT, bool N2S>
hipError_t launch_resident_grid(const ResidentParams &p, int grid, hipStream_t s, bool most, bool &done) {
  constexpr auto Kernel = search_resident<KPL, M, HT, N2S>;
  int slots = 0;
  constexpr uint32_t kLds = ResidentLds<KPL, M, HT, N2S>::kLaunchBytes;
  const hipError_t e = resident_slots<Kernel, M::grid_waves_per_simd(KPL, HT::kWords), kLds>(slots);
  if (e != hipSuccess) return e;
  done = !most || p.nq <= (uint32_t)slots;
  if (!done) return hipSuccess;
  Kernel<<<std::min(grid, slots), kWave, kLds, s>>>(p);
  return hipGetLastError();
}

template <int KPL, class M, bool N2S>
hipError_t resident_t(const ResidentParams &p, int grid, hipStream_t s) {
  using Small = VisitedLds16<M::ht_log2(KPL)>;
  using Few = VisitedLds16<M::few_ht_log2(KPL)>;
  bool done = false;
  if constexpr (Few::kWords != Small::kWords) {
    if (p.n <= Few::kMaxId) {
      const hipError_t e = launch_resident_grid<KPL, M, Few, N2S>(p, grid, s, true, done);
      if (done || e != hipSuccess) return e;
    }
  }
  if (p.n <= Small::kMaxId) return launch_resident_grid<KPL, M, Small, N2S>(p, grid, s, false, done);
  return launch_resident_grid<KPL, M, ResidentHtLarge, N2S>(p, grid, s, false, done);
}

// Small batches: a team of waves per query while the chip holds all of them at
// once.  Past that a batch's last teams wait for slots that a wave each would
// have filled.  With one frontier register the two are within 6% there for
// uint8 (1M x 128, L=64, 2,048 queries, where 1,280 fit: 246 us with teams, 259
// without), and teams have 0.85 of the speed for 96 floats (200k, L=32, beams of
// 512 ids, 2,048 queries); with more registers they fall to half (200k x 128
// uint8, L=128, beams of 512 ids, where 512 fit: 1,024 queries 0.83 of the
// speed, 2,048 0.57).
//
// Waves of a team, from the ids of a beam (W R): enough for its 64s of
// candidates, and 8 past 256 where frontiers are long.  A wave without
// candidates still crosses four barriers an iteration and repeats every merge,
// and its place could hold another team.  200k nodes, L=200, teams of 8
// against the width here, speed at 1 / 512 / 1,024 queries: 128-byte uint8, up
// to 64 ids 1.11 / 1.29 / 1.12, 128 ids 1.10 / 1.24 / 1.22, 256 ids 1.06 / 1.26 /
// 1.05; 96 floats 1.06 / 1.01 / 1.01, 1.05 / 1.17 / 1.15, 1.02 / 1.32 / 1.00.
// Two waves also where 64 ids would fit one: 1.04 to 1.23 times the speed of a
// wave per query (one query).
constexpr int team_width(uint32_t beam_ids, int most) {
  return beam_ids <= 2 * kWave ? 2 : beam_ids <= 4 * kWave ? 4 : most;
}

template <int KPL, class M, int T>
hipError_t team_t(const ResidentParams &p, hipStream_t s, bool &done) {
  constexpr auto Kernel = search_team<KPL, M, VisitedLds16<M::team_ht_log2(KPL)>, T>;
  static int slots = 0;  // per kernel
  if (slots == 0) {
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(Kernel), T * kWave, 0);
    if (e != hipSuccess) return e;
    slots = std::max(1, cus * per_cu);
  }
  done = p.nq <= (uint32_t)slots && p.n <= VisitedLds16<M::team_ht_log2(KPL)>::kMaxId;
  if (!done) return hipSuccess;
  Kernel<<<p.nq, T * kWave, 0, s>>>(p);
  return hipGetLastError();
}

template <int KPL, class M>
hipError_t team_of_width(const ResidentParams &p, hipStream_t s, bool &done) {
  const int width = team_width(p.W * p.R, M::team_waves(KPL));
  if (width == 2) return team_t<KPL, M, 2>(p, s, done);
  if constexpr (M::team_waves(KPL) > 4)
    if (width > 4) return team_t<KPL, M, M::team_waves(KPL)>(p, s, done);
  return team_t<KPL, M, 4>(p, s, done);
}

// frontier slots per lane (L <= 64 KPL)
template <class M>
hipError_t team(const ResidentParams &p, hipStream_t s, bool &done) {
  if (p.L <= 64) return team_of_width<1, M>(p, s, done);
  if (p.L <= 128) return team_of_width<2, M>(p, s, done);
  return team_of_width<4, M>(p, s, done);
}

// frontier slots per lane (L <= 64 KPL) and node_to_slot presence
template <class M>
hipError_t resident(const ResidentParams &p, int grid, hipStream_t s) {
  if constexpr (M::kStream || M::kGathered) {
    bool done = false;
    const hipError_t e = team<M>(p, s, done);
    if (done || e != hipSuccess) return e;
  }
  if constexpr (M::kLocators) {  // identity placement only
    if (p.L <= 64) return resident_t<1, M, false>(p, grid, s);
    if (p.L <= 128) return resident_t<2, M, false>(p, grid, s);
    return resident_t<4, M, false>(p, grid, s);
  } else {
    const bool n2s = p.geom.node_to_slot != nullptr;
    if (p.L <= 64) return n2s ? resident_t<1, M, true>(p, grid, s) : resident_t<1, M, false>(p, grid, s);
    if (p.L <= 128) return n2s ? resident_t<2, M, true>(p, grid, s) : resident_t<2, M, false>(p, grid, s);
    return n2s ? resident_t<4, M, true>(p, grid, s) : resident_t<4, M, false>(p, grid, s);
  }
}

template <int KPL, class M, bool N2S>
hipError_t paged_t(const PagedParams &pp, int grid, hipStream_t s) {
  const size_t lds = pp.oversub * sizeof(QSlot<KPL>);
  auto k = search_paged<KPL, M, N2S>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  k<<<grid, kWave, lds, s>>>(pp);
  return hipGetLastError();
}

template <class M>
hipError_t paged(const PagedParams &pp, int grid, hipStream_t s) {
  const bool n2s = pp.geom.node_to_slot != nullptr;
  if (pp.L <= 64) return n2s ? paged_t<1, M, true>(pp, grid, s) : paged_t<1, M, false>(pp, grid, s);
  if (pp.L <= 128) return n2s ? paged_t<2, M, true>(pp, grid, s) : paged_t<2, M, false>(pp, grid, s);
  return n2s ? paged_t<4, M, true>(pp, grid, s) : paged_t<4, M, false>(pp, grid, s);
}

template <int KPL, class M, bool N2S>
hipError_t rounds_t(const PagedParams &pp, const RoundParams &rp, int grid, hipStream_t s) {
  paged_round<KPL, M, N2S><<<grid, kWave, sizeof(QSlot<KPL>), s>>>(pp, rp);
  return hipGetLastError();
}

template <class M>
hipError_t rounds(const PagedParams &pp, const RoundParams &rp, int grid, hipStream_t s) {
  const bool n2s = pp.geom.node_to_slot != nullptr;
  if (pp.L <= 64) return n2s ? rounds_t<1, M, true>(pp, rp, grid, s) : rounds_t<1, M, false>(pp, rp, grid, s);
  if (pp.L <= 128) return n2s ? rounds_t<2, M, true>(pp, rp, grid, s) : rounds_t<2, M, false>(pp, rp, grid, s);
  return n2s ? rounds_t<4, M, true>(pp, rp, grid, s) : rounds_t<4, M, false>(pp, rp, grid, s);
}

}  // namespace detail
}  // namespace gorio
