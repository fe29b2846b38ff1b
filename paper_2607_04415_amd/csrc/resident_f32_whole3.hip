// Resident search kernels for float32 rows of 3 whole lines (96 floats).
#include "launch.hpp"

namespace gorio {

hipError_t launch_resident_f32_whole3(const ResidentParams &p, int grid, hipStream_t s) {
  return detail::resident<MetricF32Lines<3, true>>(p, grid, s);
}

}  // namespace gorio
