// What one grid dimension holds: HIP takes workgroups times threads below 2^32.
// Plain C++, so that it can be checked on the host.
#pragma once

#include <algorithm>
#include <cstdint>

namespace opscale {

// Workgroups of 256 threads, and of 64.
constexpr int64_t kMaxGrid256 = ((int64_t)1 << 24) - 1, kMaxGrid64 = ((int64_t)1 << 26) - 1;

// M rows, rows_per_wg to a workgroup of 256 threads, in as few launches as they
// take: launch(first row, rows, workgroups) for each, until one returns an error
// (not 0).
template <class F>
auto launch_rows(int64_t M, int rows_per_wg, F&& launch) {
  const int64_t most = kMaxGrid256 * rows_per_wg;
  auto e = launch((int64_t)0, std::min(M, most), (uint32_t)((std::min(M, most) + rows_per_wg - 1) / rows_per_wg));
  for (int64_t m = most; m < M && !e; m += most) {
    const int64_t rows = std::min(M - m, most);
    e = launch(m, rows, (uint32_t)((rows + rows_per_wg - 1) / rows_per_wg));
  }
  return e;
}

}  // namespace opscale
