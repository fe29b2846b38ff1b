// Resident search kernels for float32 rows of 2 lines.
#include "launch.hpp"

namespace gorio {

template <int J>
hipError_t launch_resident_f32_lines(const ResidentParams &p, int grid, hipStream_t s);

template <>
hipError_t launch_resident_f32_lines<2>(const ResidentParams &p, int grid, hipStream_t s) {
  if (p.D == 64) return detail::resident<MetricF32Lines<2, true>>(p, grid, s);
  return detail::resident<MetricF32Lines<2>>(p, grid, s);
}

}  // namespace gorio
