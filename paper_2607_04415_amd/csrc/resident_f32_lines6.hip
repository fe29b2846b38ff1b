// Resident search kernels for float32 rows of 6 lines.
#include "launch.hpp"

namespace gorio {

template <int J>
hipError_t launch_resident_f32_lines(const ResidentParams &p, int grid, hipStream_t s);

template <>
hipError_t launch_resident_f32_lines<6>(const ResidentParams &p, int grid, hipStream_t s) {
  if (p.D == 192) return detail::resident<MetricF32Lines<6, true>>(p, grid, s);
  return detail::resident<MetricF32Lines<6>>(p, grid, s);
}

}  // namespace gorio
