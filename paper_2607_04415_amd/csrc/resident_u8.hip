// Resident search kernels for uint8 rows.
#include "launch.hpp"

namespace gorio {

hipError_t launch_resident_u8_rows(const ResidentParams &p, int grid, hipStream_t s);  // resident_u8_rows.hip

// 128-d rows on 16-byte starts with the identity placement keep candidates as
// 16-byte locators.  Other rows from 36 to 256 bytes, arrangements and
// placements stream 16-byte units; rows of up to 32 bytes are one dword per
// lane, and rows past 256 bytes (whose two chunks would not fit the registers)
// take batches of 16 dwords per lane.
hipError_t launch_resident_u8(const ResidentParams &p, int grid, hipStream_t s) {
  if (p.D == 128 && p.geom.units16 != 0 && p.geom.node_to_slot == nullptr)
    return detail::resident<MetricU8<4, true, true>>(p, grid, s);
  if (p.D <= 32) return detail::resident<MetricU8<1, false>>(p, grid, s);
  if (p.D <= 256) return launch_resident_u8_rows(p, grid, s);
  return detail::resident<MetricU8<16, false>>(p, grid, s);
}

}  // namespace gorio
