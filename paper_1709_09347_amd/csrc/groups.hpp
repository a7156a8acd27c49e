// Energies whose Hankel SVDs run side by side (plain C++, used by the extraction and compiled on its own
// by a CPU test).
#pragma once

#include <algorithm>
#include <cstdint>

namespace cbs {

// Bytes that an energy of a group holds: its moments (0 where they are there anyway) and the n x n arrays of
// the SVD (both Hankel matrices, the right vectors, the rotated factor and its copy).
inline double svd_energy_bytes(double moment_bytes, int32_t n) { return moment_bytes + 5.0 * 16.0 * n * n; }

// Up to 32 energies and 64 MiB of moments.  The batch was sized by `budget`, most of the memory that was free,
// so the group keeps to a quarter of it: less than what the batch left, however little that is.
inline int32_t svd_group_size(int32_t ne, double moment_bytes, int32_t n, double budget) {
  const double most = std::min({32.0, 64.0 * (1 << 20) / std::max(moment_bytes, 1.0),
                                0.25 * budget / svd_energy_bytes(moment_bytes, n)});
  return std::max(1, std::min(ne, (int32_t)most));
}

}  // namespace cbs
