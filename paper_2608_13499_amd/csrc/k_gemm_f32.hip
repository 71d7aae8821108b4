// fp32 linear layers y[M,N] = x[M,K] W[N,K]^T (+ bias) on the fp32 matrix
// instruction v_mfma_f32_32x32x2_f32 (exact fp32 products, fp32 sums; twice
// the rate of unpacked vector FMAs).
//
// W is the MFMA "A" operand and x the "B" operand, as in the bf16 kernels: an
// accumulator lane owns one output row m and runs of four columns n.  A lane
// reads 16 bytes (four k) of its row and feeds them to four MFMAs: MFMA e of a
// chunk pair takes k = 8 c + e from lanes 0-31 and k = 8 c + 4 + e from lanes
// 32-63, the same relabelling of the summed index on both operands.
//
// Two kernels:
//  * small: a 32x32 tile per workgroup, K split over its four waves in blocks
//    of 32, operands straight into registers, the four partial tiles summed in
//    wave order through LDS.  For layers that give few larger tiles: what
//    bounds those is the chain of loads and MFMAs along K, which this cuts to
//    a quarter, and the number of workgroups;
//  * large: a 128x128 tile of four 64x64 waves, 32-wide K slices staged in LDS
//    (two stages of 32 KB, two workgroups per CU).  A slice is 64 MFMAs of 64
//    cycles per wave against 16 LDS reads: the matrix cores bound it.
#include <algorithm>

#include "common.h"
#include "launch.h"

namespace opscale {

namespace {

__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(f32x4, buffer_load16(r, off));
}

// grid.x covers N, grid.y strides over M in tiles of 32.
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(const float* __restrict__ x, const float* __restrict__ W,
                                                             const float* __restrict__ bias, float* __restrict__ y,
                                                             int M, int N, int K) {
  constexpr int kPad = 36;  // floats per LDS row: 16-byte rows, spread over the banks
  __shared__ __attribute__((aligned(16))) float red[4][32][kPad];
  const int lane = threadIdx.x & 63, fr = lane & 31, fh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n0 = blockIdx.x * 32;
  const __amdgpu_buffer_rsrc_t wr =
      make_rsrc(W + (int64_t)n0 * K, (uint32_t)((int64_t)min(32, N - n0) * K * 4));
  const uint32_t row = (uint32_t)fr * (uint32_t)K * 4u;
  const int nblk = (K + 31) / 32;
  for (int m0 = blockIdx.y * 32; m0 < M; m0 += gridDim.y * 32) {
    const __amdgpu_buffer_rsrc_t xr =
        make_rsrc(x + (int64_t)m0 * K, (uint32_t)((int64_t)min(32, M - m0) * K * 4));
    f32x4 a[2][4], b[2][4];
    // block blk: this lane's chunks 2 c + fh (c = 0..3) of 32 k; zeros past K
    auto load = [&](int blk, int buf) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int k = blk * 32 + (2 * c + fh) * 4;
        const uint32_t off = k < K ? row + (uint32_t)k * 4u : kOobOffset;
        a[buf][c] = load4(wr, off);
        b[buf][c] = load4(xr, off);
      }
    };
    f32x16 acc = {};
    auto mma = [&](int buf) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[buf][c][e], b[buf][c][e], acc, 0, 0, 0);
    };
    // (a block past the end reads zeros: no branch around the loads)
    load(wave, 0);
    for (int blk = wave; blk < nblk; blk += 8) {
      load(blk + 4, 1);
      __builtin_amdgcn_sched_barrier(0);  // (the loads stay ahead of the MFMAs)
      mma(0);
      load(blk + 8, 0);
      __builtin_amdgcn_sched_barrier(0);
      mma(1);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4*>(&red[wave][fr][g * 8 + fh * 4]) =
          f32x4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    __syncthreads();
    const int m = threadIdx.x >> 3, n = (threadIdx.x & 7) * 4;
    if (m0 + m < M && n0 + n < N) {
      f32x4 s = *reinterpret_cast<const f32x4*>(&red[0][m][n]);
#pragma unroll
      for (int w = 1; w < 4; ++w) s += *reinterpret_cast<const f32x4*>(&red[w][m][n]);
      if (bias) s += *reinterpret_cast<const f32x4*>(bias + n0 + n);
      *reinterpret_cast<f32x4*>(y + (int64_t)(m0 + m) * N + n0 + n) = s;
    }
    __syncthreads();  // the next tile reuses the LDS
  }
}

constexpr int kBM = 128, kBN = 128, kBK = 32;      // tile, and slice (128-byte rows)
constexpr int kStageBytes = (kBM + kBN) * kBK * 4;  // 32 KB
constexpr int kGroupM = 8;                          // tile-rows that sweep the tile-columns together

__global__ __launch_bounds__(256, 2) void gemm_f32_large_kernel(const float* __restrict__ x,
                                                                const float* __restrict__ W,
                                                                const float* __restrict__ bias,
                                                                float* __restrict__ y, int M, int N, int K) {
  __shared__ __attribute__((aligned(16))) char smem_raw[2 * kStageBytes];
  OPS_LDS char* smem = (OPS_LDS char*)smem_raw;
  const int tiles_m = (M + kBM - 1) / kBM, tiles_n = (N + kBN - 1) / kBN;
  const uint32_t tid = xcd_remap(blockIdx.x, gridDim.x);
  const int first = (int)(tid / (kGroupM * tiles_n)) * kGroupM, rows = min(kGroupM, tiles_m - first);
  const int in = (int)(tid % (kGroupM * tiles_n));
  const int m0 = (first + in % rows) * kBM, n0 = (in / rows) * kBN;

  const int lane = threadIdx.x & 63, fr = lane & 31, fh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(x + (int64_t)m0 * K, (uint32_t)((int64_t)min(kBM, M - m0) * K * 4));
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(W + (int64_t)n0 * K, (uint32_t)((int64_t)min(kBN, N - n0) * K * 4));

  // 16-byte chunk c of LDS row r sits at c ^ ((r / 2) mod 8): the 16 lanes of
  // a read pass (rows of one parity of bits 2..4 at one chunk) then hit 16
  // distinct bank groups.
  auto load = [&](int kt, int stage) {
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const int grp = (g & 3) * 4 + wave;  // 8 rows of x (g < 4) or W
      const int r = grp * 8 + (lane >> 3);
      const int k = kt * kBK + (((lane & 7) ^ ((r >> 1) & 7)) << 2);
      const uint32_t off = k < K ? (uint32_t)r * (uint32_t)K * 4u + (uint32_t)k * 4u : kOobOffset;
      buffer_load16_lds<kNoL1>(g < 4 ? xr : wr, smem + stage * kStageBytes + (g < 4 ? 0 : kBM * 128) + grp * 1024, off);
    }
  };
  f32x16 acc[2][2] = {};
  const int nk = (K + kBK - 1) / kBK;
  load(0, 0);
  for (int kt = 0; kt < nk; ++kt) {
    wait_vmem();
    __syncthreads();  // slice kt has landed, and every wave is done with the other stage
    if (kt + 1 < nk) load(kt + 1, (kt + 1) & 1);
    const OPS_LDS char* st = smem + (kt & 1) * kStageBytes;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      f32x4 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int rx = wm * 64 + i * 32 + fr, rw = wn * 64 + i * 32 + fr;
        b[i] = *reinterpret_cast<const OPS_LDS f32x4*>(st + rx * 128 + (((2 * c + fh) ^ ((rx >> 1) & 7)) << 4));
        a[i] = *reinterpret_cast<const OPS_LDS f32x4*>(st + kBM * 128 + rw * 128 +
                                                       (((2 * c + fh) ^ ((rw >> 1) & 7)) << 4));
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int m = m0 + wm * 64 + j * 32 + fr;
    if (m >= M) continue;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n = n0 + wn * 64 + i * 32 + g * 8 + fh * 4;
        if (n >= N) continue;
        f32x4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        if (bias) v += *reinterpret_cast<const f32x4*>(bias + n);
        *reinterpret_cast<f32x4*>(y + (int64_t)m * N + n) = v;
      }
  }
}

// From three quarters of the CUs' number of large tiles on, the large kernel
// (us, small / large: 96 tiles 1000 x 1536 x 1536 69 / 100; 288 tiles 1024 x
// 4608 x 1536 204 / 184 and 2048 x 2304 x 768 102 / 97; 4096^3 1830 / 970, 142
// TFLOP/s).  128 x 768 x 256 takes 5.0 us in the small one, 20 in the large
// and took 26 in the 64x64 vector-FMA tile used before.
constexpr int64_t kF32LargeTiles = 192;

}  // namespace

hipError_t launch_linear_f32(const void* x, const void* W, const void* bias, void* y, int64_t M, int64_t N, int64_t K,
                             hipStream_t s) {
  const auto* xf = static_cast<const float*>(x);
  const auto* wf = static_cast<const float*>(W);
  const auto* bf = static_cast<const float*>(bias);
  auto* yf = static_cast<float*>(y);
  const int64_t tiles = ((M + kBM - 1) / kBM) * ((N + kBN - 1) / kBN);
  if (tiles >= kF32LargeTiles) {
    hipLaunchKernelGGL(gemm_f32_large_kernel, dim3((unsigned)tiles), dim3(256), 0, s, xf, wf, bf, yf, (int)M, (int)N,
                       (int)K);
  } else {
    hipLaunchKernelGGL(gemm_f32_small_kernel,
                       dim3((unsigned)((N + 31) / 32), (unsigned)std::min<int64_t>(65535, (M + 31) / 32)), dim3(256), 0,
                       s, xf, wf, bf, yf, (int)M, (int)N, (int)K);
  }
  return hipGetLastError();
}

}  // namespace opscale
