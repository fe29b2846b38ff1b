// Resident search kernels for float32 rows of at most 8 floats.
#include "launch.hpp"

namespace gorio {

hipError_t launch_resident_f32_own(const ResidentParams &p, int grid, hipStream_t s) {
  return detail::resident<MetricF32Own>(p, grid, s);
}

}  // namespace gorio
