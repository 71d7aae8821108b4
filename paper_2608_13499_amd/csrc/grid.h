// What one grid dimension holds: HIP takes workgroups times threads below 2^32.
// Plain C++, so that it can be checked on the host.
#pragma once

#include <cstdint>

namespace opscale {

// Workgroups of 256 threads, and of 64.
constexpr int64_t kMaxGrid256 = ((int64_t)1 << 24) - 1, kMaxGrid64 = ((int64_t)1 << 26) - 1;

}  // namespace opscale
