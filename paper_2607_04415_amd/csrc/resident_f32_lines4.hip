// Resident search kernels for float32 rows of 4 lines.
#include "launch.hpp"

namespace gorio {

template <int J>
hipError_t launch_resident_f32_lines(const ResidentParams &p, int grid, hipStream_t s);

template <>
hipError_t launch_resident_f32_lines<4>(const ResidentParams &p, int grid, hipStream_t s) {
  if (p.D == 128) return detail::resident<MetricF32Lines<4, true>>(p, grid, s);
  return detail::resident<MetricF32Lines<4>>(p, grid, s);
}

}  // namespace gorio
