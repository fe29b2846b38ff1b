// Resident search kernels for float32 rows: two variants per number of 128-byte
// lines a row takes (D <= 256), whole lines (D a multiple of 32) and a ragged
// last one, each number in a translation unit of its own
// (resident_f32_lines*.hip), so that they compile in parallel.  Whole lines
// need no test of what a block holds, which lets the sums overlap the LDS
// passes: 100k nodes, R=64, W=8, 5,000 queries, us a call with the ragged
// variant / the whole one: 32 floats, L=64 535 / 467, L=200 1,555 / 1,352; 64
// 736 / 676, 1,956 / 1,794; 128 1,267 / 1,210, 3,591 / 3,321; 160 1,946 /
// 1,829, 4,862 / 4,533; 256 2,896 / 2,742, 7,047 / 6,648.
#include "launch.hpp"

namespace gorio {

template <int J>
hipError_t launch_resident_f32_lines(const ResidentParams &p, int grid, hipStream_t s);

hipError_t launch_resident_f32_own(const ResidentParams &p, int grid, hipStream_t s);  // resident_f32_own.hip

hipError_t launch_resident_f32(const ResidentParams &p, int grid, hipStream_t s) {
  if (p.D <= 8) return launch_resident_f32_own(p, grid, s);
  switch ((p.D + 31) / 32) {
    case 1: return launch_resident_f32_lines<1>(p, grid, s);
    case 2: return launch_resident_f32_lines<2>(p, grid, s);
    case 3: return launch_resident_f32_lines<3>(p, grid, s);
    case 4: return launch_resident_f32_lines<4>(p, grid, s);
    case 5: return launch_resident_f32_lines<5>(p, grid, s);
    case 6: return launch_resident_f32_lines<6>(p, grid, s);
    case 7: return launch_resident_f32_lines<7>(p, grid, s);
    default: return launch_resident_f32_lines<8>(p, grid, s);
  }
}

}  // namespace gorio
