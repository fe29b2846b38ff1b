// Resident search kernels for uint8 rows in 16-byte units.
#include "launch.hpp"

namespace gorio {

hipError_t launch_resident_u8_rows(const ResidentParams &p, int grid, hipStream_t s) {
  if (p.D == 128) return detail::resident<MetricU8Rows<1, true>>(p, grid, s);
  if (p.D < 128) return detail::resident<MetricU8Rows<1, false>>(p, grid, s);
  return detail::resident<MetricU8Rows<2, false>>(p, grid, s);
}

}  // namespace gorio
