// What one grid dimension holds: HIP takes workgroups times threads below 2^32.
// Plain C++, so that it can be checked on the host.
#pragma once

#include <algorithm>
#include <cstdint>

namespace opscale {

// Workgroups of 256 threads, and of 64.
constexpr int64_t kMaxGrid256 = ((int64_t)1 << 24) - 1, kMaxGrid64 = ((int64_t)1 << 26) - 1;

// Norms on a share of the CUs: a workgroup per row brings its CU fewer bytes at a time
// than four waves of a row each, which shows on few CUs with rows enough to fill them
// (measured on 26, 64, 128 and 154; on 192 and more it is equal or slower).
//
// RMS Norm, of `nvec` 16-byte vectors a row (us, workgroup / wave a row: 8871 rows of
// 8192 on 128 CUs 74.0 / 63.9, on 154 76.6 / 63.9, on 192 54.0 / 53.5; 1023 of 4096 on 64
// 10.5 / 10.2; 1023 of 1536 on 64 7.2 / 6.4; with little to do, 256 of 8192 on 128, 6.7 /
// 7.8).  Rows past 16 vectors a lane would be read twice (1023 of 16384 on 64 32.0 /
// 37.9).
constexpr int64_t kWaveRowsFill = 20480, kAddWaveRowsFill = 40960;  // elements a CU
inline bool rmsnorm_wave_rows(int64_t M, int64_t H, int64_t nvec, int cus) {
  return cus <= 160 && nvec <= 16 * 64 && M * H >= kWaveRowsFill * cus;
}

// Residual norm, whose wave holds a row in fp32 and loads it piece by piece, so needs
// more rows to be full (8871 of 4096 on 64 CUs 117 / 106, in fp32 227 / 194; 2048 of 1536
// on 64 13.0 / 11.6; 1023 of 4096 on 128, eight a CU, 11.5 / 14.7).  Past 4096 a lane has
// too many registers (8871 of 8192 on 64 235 / 390).
inline bool add_rmsnorm_wave_rows(int64_t M, int64_t H, int cus) {
  return cus <= 160 && H <= 4096 && M * H >= kAddWaveRowsFill * cus;
}

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
