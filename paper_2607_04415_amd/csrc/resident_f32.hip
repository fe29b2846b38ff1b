// Resident search kernels for float32 rows: one variant per number of 128-byte
// lines a row takes (D <= 256), each in a translation unit of its own
// (resident_f32_lines*.hip), so that they compile in parallel.
#include "launch.hpp"

namespace gorio {

template <int J>
hipError_t launch_resident_f32_lines(const ResidentParams &p, int grid, hipStream_t s);

hipError_t launch_resident_f32_whole3(const ResidentParams &p, int grid, hipStream_t s);

hipError_t launch_resident_f32(const ResidentParams &p, int grid, hipStream_t s) {
  switch ((p.D + 31) / 32) {
    case 1: return launch_resident_f32_lines<1>(p, grid, s);
    case 2: return launch_resident_f32_lines<2>(p, grid, s);
    case 3:
      // whole lines: the ragged line's tests cost a kernel with one wave per
      // SIMD its overlap (1M x 96, L=128, W=8, 10k queries: 4.83 against 4.18 ms)
      if (p.D == 96) return launch_resident_f32_whole3(p, grid, s);
      return launch_resident_f32_lines<3>(p, grid, s);
    case 4: return launch_resident_f32_lines<4>(p, grid, s);
    case 5: return launch_resident_f32_lines<5>(p, grid, s);
    case 6: return launch_resident_f32_lines<6>(p, grid, s);
    case 7: return launch_resident_f32_lines<7>(p, grid, s);
    default: return launch_resident_f32_lines<8>(p, grid, s);
  }
}

}  // namespace gorio
