// Bandwidth-bound operators: RMS Norm and the fused SiLU-multiply (SwiGLU).
//
// Both stream their operands once from HBM with 16-byte loads and stores per
// lane, keep the math in fp32 and round once at the output.
#include "common.h"
#include "grid.h"
#include "launch.h"

namespace opscale {

// ------------------------------------------------------------- RMS Norm ----
// WPR waves per row: the workgroup's four, or one for short rows.  VPL = 16-byte
// vectors per lane held in registers (a row of up to VPL*WPR*64*16 bytes is
// read once); VPL == 0 selects the streaming variant for longer rows, which
// reads the row a second time (from L2) to normalize.
template <bool BF16, int VPL, int WPR>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const void* x, const void* __restrict__ w,
                                                      void* y, int64_t M,
                                                      int H, float eps) {
  constexpr int EPV = BF16 ? 8 : 4;  // elements per 16-byte vector
  constexpr int STEP = 64 * WPR;
  const int lane = threadIdx.x & (STEP - 1);  // lane of the row
  const int64_t row = (int64_t)blockIdx.x * (4 / WPR) + threadIdx.x / STEP;
  if (row >= M) return;
  const int nvec = H / EPV;
  const u32x4* xr = reinterpret_cast<const u32x4*>(static_cast<const char*>(x) + row * (int64_t)H * (BF16 ? 2 : 4));
  u32x4* yr = reinterpret_cast<u32x4*>(static_cast<char*>(y) + row * (int64_t)H * (BF16 ? 2 : 4));
  const u32x4* wr = reinterpret_cast<const u32x4*>(w);

  auto sq = [](const u32x4& v) {
    float s = 0.f;
    if constexpr (BF16) {
      const uint32_t a[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float lo = bf_lo(a[i]), hi = bf_hi(a[i]);
        s = fmaf(lo, lo, s);
        s = fmaf(hi, hi, s);
      }
    } else {
      const float a[4] = {__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]),
                          __uint_as_float(v[3])};
#pragma unroll
      for (int i = 0; i < 4; ++i) s = fmaf(a[i], a[i], s);
    }
    return s;
  };
  auto scale = [](const u32x4& v, const u32x4& g, float r) {
    u32x4 o;
    if constexpr (BF16) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = pack_bf2(bf_lo(v[i]) * r * bf_lo(g[i]), bf_hi(v[i]) * r * bf_hi(g[i]));
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = __float_as_uint(__uint_as_float(v[i]) * r * __uint_as_float(g[i]));
    }
    return o;
  };

  float ss = 0.f;
  if constexpr (VPL > 0) {
    // the row and the weight are requested together, so the weight (an L2
    // hit) costs no round trip after the reduction.  Plain (cached) loads and
    // stores: measured 1-2 us faster on an 8871 x 4096 row block than the
    // nontemporal forms, and faster than a device copy of the same bytes.
    u32x4 v[VPL], g[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int idx = lane + i * STEP;
      v[i] = idx < nvec ? xr[idx] : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int idx = lane + i * STEP;
      g[i] = idx < nvec ? wr[idx] : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i) ss += sq(v[i]);
    ss = row_sum<WPR>(ss);
    const float r = rsqrtf(ss / (float)H + eps);
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int idx = lane + i * STEP;
      if (idx < nvec) yr[idx] = scale(v[i], g[i], r);
    }
  } else {
    for (int idx = lane; idx < nvec; idx += STEP) ss += sq(xr[idx]);
    ss = row_sum<WPR>(ss);
    const float r = rsqrtf(ss / (float)H + eps);
    for (int idx = lane; idx < nvec; idx += STEP) yr[idx] = scale(xr[idx], wr[idx], r);
  }
}

template <bool BF16, int WPR>
static hipError_t rmsnorm_dispatch(const void* x, const void* w, void* y, int64_t M, int64_t H,
                                   float eps, hipStream_t s) {
  constexpr int kRows = 4 / WPR;  // rows of a workgroup
  const int64_t nvec = H / (BF16 ? 8 : 4);
  const int vpl = (int)((nvec + 64 * WPR - 1) / (64 * WPR));
  const int h = (int)H;
  const int64_t row_bytes = H * (BF16 ? 2 : 4);
  return launch_rows(M, kRows, [&](int64_t m, int64_t rows, uint32_t grid) {
    const char* xm = static_cast<const char*>(x) + m * row_bytes;
    char* ym = static_cast<char*>(y) + m * row_bytes;
#define OPS_RMS(V) \
  hipLaunchKernelGGL((rmsnorm_kernel<BF16, V, WPR>), dim3(grid), dim3(256), 0, s, xm, w, ym, rows, h, eps)
    if (vpl <= 1) OPS_RMS(1);
    else if (vpl <= 2) OPS_RMS(2);
    else if (vpl <= 4) OPS_RMS(4);
    else if (vpl <= 8) OPS_RMS(8);
    else if (vpl <= 16) OPS_RMS(16);
    else if constexpr (WPR > 1) OPS_RMS(0);
#undef OPS_RMS
    return hipGetLastError();
  });
}

hipError_t launch_rmsnorm(const void* x, const void* w, void* y, int64_t M, int64_t H, float eps,
                          bool bf16, hipStream_t s) {
  // rows of up to 255 vectors leave part of a workgroup idle, which shows where
  // there are rows enough to fill the chip with a wave each (us, wave / workgroup a
  // row: 1032 wide, 1023 rows 3.27 / 3.27, 2048 4.0 / 4.2, 8871 10.0 / 12.0; 1536
  // wide, 100 rows 2.57 / 2.44, 20000 22.8 / 24.1; 2048 wide, 20000 30.0 / 29.6)
  const int64_t nvec = H / (bf16 ? 8 : 4);
  // (too little for one CU: its calls are spared the 0.3 us that the mask's query takes)
  const bool wave = nvec <= kWaveRowMaxVec || (nvec < 256 && M >= 2048) ||
                    (M * H >= kWaveRowsFill && rmsnorm_wave_rows(M, H, nvec, stream_cus(s)));
  if (!wave)
    return bf16 ? rmsnorm_dispatch<true, 4>(x, w, y, M, H, eps, s) : rmsnorm_dispatch<false, 4>(x, w, y, M, H, eps, s);
  return bf16 ? rmsnorm_dispatch<true, 1>(x, w, y, M, H, eps, s) : rmsnorm_dispatch<false, 1>(x, w, y, M, H, eps, s);
}

// --------------------------------------------------------------- SwiGLU ----
// grid.x covers one row's 16-byte output vectors (256 threads x VPT vectors
// each), grid.y strides over rows.  STREAM: nontemporal accesses, for batches
// that do not stay in the caches between the projections around this anyway.
template <bool BF16, int VPT, bool STREAM>
__global__ __launch_bounds__(256) void swiglu_kernel(const void* __restrict__ gu, void* __restrict__ out,
                                                     int64_t M, int64_t F) {
  constexpr int EPV = BF16 ? 8 : 4;
  constexpr int ES = BF16 ? 2 : 4;
  const int64_t nvec = F / EPV;
  for (int64_t row = blockIdx.y; row < M; row += gridDim.y) {
    const u32x4* g = reinterpret_cast<const u32x4*>(static_cast<const char*>(gu) + row * 2 * F * ES);
    const u32x4* u = reinterpret_cast<const u32x4*>(static_cast<const char*>(gu) + (row * 2 * F + F) * ES);
    u32x4* o = reinterpret_cast<u32x4*>(static_cast<char*>(out) + row * F * ES);
    u32x4 gv[VPT], uv[VPT];
    const int64_t base = (int64_t)blockIdx.x * 256 * VPT + threadIdx.x;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int64_t idx = base + i * 256;
      if (idx < nvec) {
        gv[i] = STREAM ? __builtin_nontemporal_load(g + idx) : g[idx];
        uv[i] = STREAM ? __builtin_nontemporal_load(u + idx) : u[idx];
      }
    }
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int64_t idx = base + i * 256;
      if (idx >= nvec) continue;
      const u32x4 ga = gv[i], ua = uv[i];
      u32x4 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (BF16) {
          const float g0 = bf_lo(ga[e]), g1 = bf_hi(ga[e]);
          const float s0 = g0 / (1.f + __expf(-g0)), s1 = g1 / (1.f + __expf(-g1));
          r[e] = pack_bf2(s0 * bf_lo(ua[e]), s1 * bf_hi(ua[e]));
        } else {
          const float g0 = __uint_as_float(ga[e]);
          r[e] = __float_as_uint(g0 / (1.f + expf(-g0)) * __uint_as_float(ua[e]));
        }
      }
      if (STREAM) __builtin_nontemporal_store(r, o + idx);
      else o[idx] = r;
    }
  }
}

template <bool BF16, int VPT, bool STREAM>
static hipError_t swiglu_dispatch(const void* gu, void* out, int64_t M, int64_t F, hipStream_t s) {
  const int64_t nvec = F / (BF16 ? 8 : 4);
  const unsigned gx = (unsigned)((nvec + 256 * VPT - 1) / (256 * VPT));
  const unsigned gy = (unsigned)(M < 65535 ? M : 65535);
  hipLaunchKernelGGL((swiglu_kernel<BF16, VPT, STREAM>), dim3(gx, gy), dim3(256), 0, s, gu, out, M, F);
  return hipGetLastError();
}

hipError_t launch_swiglu(const void* gu, void* out, int64_t M, int64_t F, bool bf16, hipStream_t s) {
  // Up to 256 rows, and up to 16 million outputs of rows of 8192 and wider: cached
  // accesses and one vector a thread, i.e. twice the workgroups.  What is small
  // stays in the caches from the projection before (the first pair of each) and
  // gains by both; larger, the last-level cache evicts what the next operator
  // reads.  us, two nontemporal / one cached, operands just written | cold:
  //   F = 2560:  M = 48 2.8 / 2.4 | 3.1 / 2.4, 256 3.5 / 2.7 | 3.7 / 3.2,
  //              512 (the reverse from here) cold 4.8 / 5.2, 1023 7.1 / 8.0
  //   F = 8192:  256 4.3 / 3.6 | 4.8 / 4.4, 512 5.9 / 5.4 | 6.7 / 6.3,
  //              1023 9.4 / 9.7 | 10.9 / 11.8, 2048 17.4 / 16.3 | 19.7 / 19.6
  //   F = 14336: 256 5.7 / 4.8 | 6.5 / 5.9, 512 8.9 / 8.2 | 10.5 / 10.7,
  //              1023 16.0 / 14.5 | 17.6 / 17.7, 2048 cold 28.9 / 35.9
  //   F = 28672: 100 5.0 / 4.3 | 5.7 / 5.1, 256 8.4 / 8.0 | 9.8 / 10.7,
  //              512 15.7 / 14.8 | 17.6 / 17.6
  // Widths of 512 to 2048 differ by less than the runs; 4096 to 7168, 11008 and
  // 18944 lie between their neighbours.  Cold inputs of 6 to 16 million outputs cost
  // up to 8 % more than before, which the MLP, where they are warm, gains.
  const bool small = M * F <= ((int64_t)1 << 24) && (F >= 8192 || M <= 256);
  if (small)
    return bf16 ? swiglu_dispatch<true, 1, false>(gu, out, M, F, s) : swiglu_dispatch<false, 1, false>(gu, out, M, F, s);
  return bf16 ? swiglu_dispatch<true, 2, true>(gu, out, M, F, s) : swiglu_dispatch<false, 2, true>(gu, out, M, F, s);
}

// ---------------------------------------------------------------- flush ----
// Reads every byte of buf, so the caches then hold clean lines of buf and
// nothing of the timed operator's operands.  (A writing flush would leave the
// last-level cache full of dirty lines, and the next kernel would pay for
// their write-back.)  The XOR of the data is stored only if it equals `tag`,
// which keeps the loads alive and practically never happens.
__global__ __launch_bounds__(256) void flush_kernel(u32x4* buf, size_t nvec, uint32_t tag) {
  uint32_t h = 0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (size_t)gridDim.x * 256) {
    const u32x4 v = buf[i];  // a plain load: it allocates in L2 and the MALL
    h ^= v[0] ^ v[1] ^ v[2] ^ v[3];
  }
  const size_t me = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (h == tag && me < nvec) buf[me][0] = h;
}

hipError_t launch_flush(void* buf, size_t bytes, hipStream_t s) {
  const size_t nvec = bytes / 16;
  if (nvec == 0) return hipSuccess;
  hipLaunchKernelGGL(flush_kernel, dim3(2048), dim3(256), 0, s, static_cast<u32x4*>(buf), nvec,
                     0x5a5a5a5au);
  return hipGetLastError();
}

}  // namespace opscale
