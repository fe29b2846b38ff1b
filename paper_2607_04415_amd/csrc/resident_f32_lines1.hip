// Resident search kernels for float32 rows of 1 line.
#include "launch.hpp"

namespace gorio {

template <int J>
hipError_t launch_resident_f32_lines(const ResidentParams &p, int grid, hipStream_t s);

template <>
hipError_t launch_resident_f32_lines<1>(const ResidentParams &p, int grid, hipStream_t s) {
  if (p.D == 32) return detail::resident<MetricF32Lines<1, true>>(p, grid, s);
  return detail::resident<MetricF32Lines<1>>(p, grid, s);
}

}  // namespace gorio
