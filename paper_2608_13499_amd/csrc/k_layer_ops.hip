// The operators around attention in a decoder layer: rotary embedding of q
// and k, the paged KV-cache write, and the residual add fused into RMS Norm.
// All three are bandwidth-bound; each moves its operands once with 8- or
// 16-byte accesses per lane and computes in fp32 (the RoPE angle in fp64).
#include <cmath>
#include <type_traits>

#include "common.h"
#include "grid.h"
#include "launch.h"

namespace opscale {

namespace {
constexpr double kTwoPi = 6.283185307179586476925286766559;
}  // namespace

// ------------------------------------------------------------------ RoPE ----
// One workgroup per token.  A thread owns 4 consecutive rotation pairs
// (i .. i + 3, partners i + D/2 .. i + D/2 + 3) of one head, q heads first
// then k heads.  The angle p * theta^(-2i/D) is formed in fp64 and reduced to
// [-pi, pi] there, so the fp32 sine and cosine see an argument accurate to
// ~1e-7 rad at any position.
// Large batches are bound by memory, one token by the chain of loads, angle and
// stores: each of the D/2 angles is computed once, by one thread, while the
// rows are on their way, rather than by every head after them (us, 32 + 8 heads
// of 128, each angle per head / once: one token 3.2 / 2.1, 256 3.9 / 2.7, 1023
// 6.3 / 4.9, 8871 36.0 / 34.2; 64 + 8 heads, one token 4.4 / 2.8).  NT: 64 threads
// a token where they hold its heads at once, 256 otherwise (us, 256 / 64 threads:
// 4 + 4 heads of 64, 20000 tokens 15.6 / 9.5; 8 + 8, 8871 11.5 / 7.8).
template <bool BF16, int D, int NT>
__global__ __launch_bounds__(NT) void rope_kernel(void* q, void* k, int64_t q_stride, int64_t k_stride,
                                                   const int32_t* __restrict__ pos, int Hq, int Hkv,
                                                   double log2_theta) {
  constexpr int HALF = D / 2, QUADS = HALF / 4, kPer = 3;  // quads of a thread requested at once
  using V = std::conditional_t<BF16, u32x2, u32x4>;
  __shared__ __attribute__((aligned(16))) float cosine[HALF], sine[HALF];
  const int64_t t = blockIdx.x;
  const int total = (Hq + Hkv) * QUADS;
  const double p = (double)pos[t];
  V lo[kPer], hi[kPer];
  auto row = [&](int idx) {
    const int head = idx / QUADS, quad = idx % QUADS;
    const int64_t e = (head < Hq ? t * q_stride + (int64_t)head * D : t * k_stride + (int64_t)(head - Hq) * D) + 4 * quad;
    return static_cast<char*>(head < Hq ? q : k) + e * (BF16 ? 2 : 4);
  };
  auto load = [&](int idx0) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (idx0 + i * NT >= total) break;
      const char* e = row(idx0 + i * NT);
      lo[i] = *reinterpret_cast<const V*>(e);
      hi[i] = *reinterpret_cast<const V*>(e + HALF * (BF16 ? 2 : 4));
    }
  };
  load(threadIdx.x);
  if (threadIdx.x < HALF) {
    const int i = threadIdx.x;
    const double ang = p * exp2(-(2.0 * i / D) * log2_theta);
    const float r = (float)(ang - kTwoPi * rint(ang * (1.0 / kTwoPi)));
    sincosf(r, &sine[i], &cosine[i]);
  }
  __syncthreads();
  for (int idx0 = threadIdx.x;;) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int idx = idx0 + i * NT;
      if (idx >= total) break;
      const f32x4 cs = *reinterpret_cast<const f32x4*>(cosine + 4 * (idx % QUADS));
      const f32x4 sn = *reinterpret_cast<const f32x4*>(sine + 4 * (idx % QUADS));
      float a[4], b[4], ra[4], rb[4];
      if constexpr (BF16) {
        a[0] = bf_lo(lo[i][0]), a[1] = bf_hi(lo[i][0]), a[2] = bf_lo(lo[i][1]), a[3] = bf_hi(lo[i][1]);
        b[0] = bf_lo(hi[i][0]), b[1] = bf_hi(hi[i][0]), b[2] = bf_lo(hi[i][1]), b[3] = bf_hi(hi[i][1]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = __uint_as_float(lo[i][j]), b[j] = __uint_as_float(hi[i][j]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ra[j] = a[j] * cs[j] - b[j] * sn[j];
        rb[j] = b[j] * cs[j] + a[j] * sn[j];
      }
      V rlo, rhi;
      if constexpr (BF16) {
        rlo = V{pack_bf2(ra[0], ra[1]), pack_bf2(ra[2], ra[3])};
        rhi = V{pack_bf2(rb[0], rb[1]), pack_bf2(rb[2], rb[3])};
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) rlo[j] = __float_as_uint(ra[j]), rhi[j] = __float_as_uint(rb[j]);
      }
      char* e = row(idx);
      *reinterpret_cast<V*>(e) = rlo;
      *reinterpret_cast<V*>(e + HALF * (BF16 ? 2 : 4)) = rhi;
    }
    idx0 += kPer * NT;
    if (idx0 >= total) break;
    load(idx0);
  }
}

hipError_t launch_rope(void* q, void* k, int64_t q_stride, int64_t k_stride, const int32_t* pos, int64_t T,
                       int32_t Hq, int32_t Hkv, int32_t D, double theta, bool bf16, hipStream_t s) {
  const double l2 = std::log2(theta);
  // (three quads a lane; the other three waves would only take up places)
  const bool one = (Hq + Hkv) * (D / 8) <= 3 * 64;
  const dim3 grid((unsigned)T);
#define OPS_ROPE(B, DD)                                                                                               \
  if (one)                                                                                                            \
    hipLaunchKernelGGL((rope_kernel<B, DD, 64>), grid, dim3(64), 0, s, q, k, q_stride, k_stride, pos, Hq, Hkv, l2);   \
  else                                                                                                                \
    hipLaunchKernelGGL((rope_kernel<B, DD, 256>), grid, dim3(256), 0, s, q, k, q_stride, k_stride, pos, Hq, Hkv, l2)
  if (bf16) {
    if (D == 128) {
      OPS_ROPE(true, 128);
    } else {
      OPS_ROPE(true, 64);
    }
  } else {
    if (D == 128) {
      OPS_ROPE(false, 128);
    } else {
      OPS_ROPE(false, 64);
    }
  }
#undef OPS_ROPE
  return hipGetLastError();
}

// ------------------------------------------------------- KV cache write ----
// The rows to copy are a list of 16-byte chunks: token t owns chunks
// [t * 2 * row_chunks, (t + 1) * 2 * row_chunks), its K row first, then its V
// row, each copied to cache row `slot` (the cache [num_blocks, block_size,
// Hkv, D] is an array of such rows).  A workgroup takes kChunksPerWg
// consecutive chunks, a thread kCwPerThread of them 256 apart: every load (the
// row chunks and their tokens' slots) is issued before the first store.
// Tokens whose slot is outside [0, num_slots) are skipped.
constexpr int kCwPerThread = 4;
constexpr int kChunksPerWg = 256 * kCwPerThread;
__global__ __launch_bounds__(256) void cache_write_kernel(const char* __restrict__ k, const char* __restrict__ v,
                                                         int64_t kv_stride_bytes, char* kc, char* vc,
                                                         const int32_t* __restrict__ slots, int row_chunks,
                                                         int64_t T, int64_t num_slots) {
  const int64_t total = T * 2 * row_chunks;
  for (int64_t blk = blockIdx.x; blk * kChunksPerWg < total; blk += gridDim.x) {
  const int64_t q0 = blk * kChunksPerWg + threadIdx.x;
  u32x4 val[kCwPerThread];
  int64_t slot[kCwPerThread];
#pragma unroll
  for (int i = 0; i < kCwPerThread; ++i) {
    const int64_t q = min(q0 + i * 256, total - 1);  // clamped: the stores below check q
    const int64_t t = q / (2 * row_chunks);
    const int c = (int)(q - t * 2 * row_chunks);
    const bool isv = c >= row_chunks;
    val[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>((isv ? v : k) + t * kv_stride_bytes) +
                                        (isv ? c - row_chunks : c));
    slot[i] = slots[t];
  }
#pragma unroll
  for (int i = 0; i < kCwPerThread; ++i) {
    const int64_t q = q0 + i * 256;
    if (q >= total || slot[i] < 0 || slot[i] >= num_slots) continue;
    const int64_t t = q / (2 * row_chunks);
    const int c = (int)(q - t * 2 * row_chunks);
    const bool isv = c >= row_chunks;
    *(reinterpret_cast<u32x4*>((isv ? vc : kc) + slot[i] * (int64_t)row_chunks * 16) + (isv ? c - row_chunks : c)) =
        val[i];
  }
  }  // block stride
}

hipError_t launch_cache_write(const void* k, const void* v, int64_t kv_stride, void* kc, void* vc,
                              const int32_t* slots, int64_t T, int32_t Hkv, int32_t D, int64_t num_slots,
                              bool bf16, hipStream_t s) {
  const int es = bf16 ? 2 : 4;
  const int row_chunks = (int)((int64_t)Hkv * D * es / 16);
  const int64_t total = T * 2 * row_chunks;
  const int64_t blocks = std::min<int64_t>((total + kChunksPerWg - 1) / kChunksPerWg, 1 << 20);
  hipLaunchKernelGGL(cache_write_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                     static_cast<const char*>(k), static_cast<const char*>(v), kv_stride * es,
                     static_cast<char*>(kc), static_cast<char*>(vc), slots, row_chunks, T, num_slots);
  return hipGetLastError();
}

// ------------------------------------------------- residual + RMS Norm ----
// WPR waves per row (the workgroup's four, or one for short rows), the row held in
// registers as fp32: r = x + residual is written back to `residual` (rounded
// once), y = r / rms(r) * w.  VPL 16-byte vectors per lane cover the row.  The
// row, the residual and w are all requested before the first store: y and
// residual may alias x as far as the compiler knows, and w read after a store
// cost a round trip per vector (H = 4096, one row 4.2 us, now 2.0; 1023 rows
// 10.7, now 7.1; 8871 rows 58.7, now 45.8).
template <bool BF16, int VPL, int WPR>
__global__ __launch_bounds__(256) void add_rmsnorm_kernel(const void* x, void* res, const void* __restrict__ w,
                                                          void* y, int64_t M, int H, float eps) {
  constexpr int EPV = BF16 ? 8 : 4;  // elements per 16-byte vector
  constexpr int STEP = 64 * WPR;
  const int lane = threadIdx.x & (STEP - 1);  // lane of the row
  const int64_t row = (int64_t)blockIdx.x * (4 / WPR) + threadIdx.x / STEP;
  if (row >= M) return;
  const int nvec = H / EPV;
  const int64_t off = row * (int64_t)H * (BF16 ? 2 : 4);
  const u32x4* xr = reinterpret_cast<const u32x4*>(static_cast<const char*>(x) + off);
  u32x4* rr = reinterpret_cast<u32x4*>(static_cast<char*>(res) + off);
  u32x4* yr = reinterpret_cast<u32x4*>(static_cast<char*>(y) + off);
  const u32x4* wr = reinterpret_cast<const u32x4*>(w);
  auto unpack = [](const u32x4& v, float* f) {
    if constexpr (BF16) {
#pragma unroll
      for (int i = 0; i < 4; ++i) f[2 * i] = bf_lo(v[i]), f[2 * i + 1] = bf_hi(v[i]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(v[i]);
    }
  };
  auto pack = [](const float* f) {
    u32x4 o;
    if constexpr (BF16) {
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = pack_bf2(f[2 * i], f[2 * i + 1]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = __float_as_uint(f[i]);
    }
    return o;
  };
  // plain (cached) loads and stores, as in the RMS Norm kernel (faster than
  // the nontemporal forms on a streamed row block)
  constexpr u32x4 kZero = {0u, 0u, 0u, 0u};
  // A wave of a long row adds as it loads and reads the weight last: fewer registers,
  // more waves (it runs where there are rows enough).
  constexpr bool kLate = WPR == 1 && VPL > 2;
  u32x4 xv[VPL], rv[VPL], g[VPL];
  float sum[VPL][EPV] = {};
  float ss = 0.f;
  auto add = [&](int i, const u32x4& xi, const u32x4& ri) {
    float a[EPV], b[EPV];
    unpack(xi, a);
    unpack(ri, b);
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
      sum[i][e] = a[e] + b[e];
      ss = fmaf(sum[i][e], sum[i][e], ss);
    }
  };
  if constexpr (kLate) {
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int idx = lane + i * STEP;
      if (idx < nvec) add(i, xr[idx], rr[idx]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int idx = lane + i * STEP;
      xv[i] = idx < nvec ? xr[idx] : kZero;
      rv[i] = idx < nvec ? rr[idx] : kZero;
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int idx = lane + i * STEP;
      g[i] = idx < nvec ? wr[idx] : kZero;
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i) add(i, xv[i], rv[i]);
  }
  ss = row_sum<WPR>(ss);
  const float r = rsqrtf(ss / (float)H + eps);
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int idx = lane + i * STEP;
    if (idx >= nvec) continue;
    rr[idx] = pack(sum[i]);
    if constexpr (kLate) g[i] = wr[idx];
    float gf[EPV], o[EPV];
    unpack(g[i], gf);
#pragma unroll
    for (int e = 0; e < EPV; ++e) o[e] = sum[i][e] * r * gf[e];
    yr[idx] = pack(o);
  }
}

template <bool BF16, int WPR>
static hipError_t add_rmsnorm_dispatch(const void* x, void* res, const void* w, void* y, int64_t M, int64_t H,
                                       float eps, hipStream_t s) {
  constexpr int kRows = 4 / WPR;  // rows of a workgroup
  const int64_t nvec = H / (BF16 ? 8 : 4);
  const int vpl = (int)((nvec + 64 * WPR - 1) / (64 * WPR));
  const int h = (int)H;
  const int64_t row_bytes = H * (BF16 ? 2 : 4);
  return launch_rows(M, kRows, [&](int64_t m, int64_t rows, uint32_t grid) {
    const char* xm = static_cast<const char*>(x) + m * row_bytes;
    char *rm = static_cast<char*>(res) + m * row_bytes, *ym = static_cast<char*>(y) + m * row_bytes;
#define OPS_ADDRMS(V) \
  hipLaunchKernelGGL((add_rmsnorm_kernel<BF16, V, WPR>), dim3(grid), dim3(256), 0, s, xm, rm, w, ym, rows, h, eps)
    if (vpl <= 1) OPS_ADDRMS(1);
    else if (vpl <= 2) OPS_ADDRMS(2);
    else if (vpl <= 4) OPS_ADDRMS(4);
    else if constexpr (WPR == 1) {  // (rows of at most 16 KB, here of 4096 elements)
      if (vpl <= 8) OPS_ADDRMS(8);
      else if constexpr (!BF16) OPS_ADDRMS(16);
    }
#undef OPS_ADDRMS
    return hipGetLastError();
  });
}

hipError_t launch_add_rmsnorm(const void* x, void* res, const void* w, void* y, int64_t M, int64_t H, float eps,
                              bool bf16, hipStream_t s) {
  const bool wave = H / (bf16 ? 8 : 4) <= kWaveRowMaxVec ||
                    (M * H >= kAddWaveRowsFill && add_rmsnorm_wave_rows(M, H, stream_cus(s)));
  if (!wave)
    return bf16 ? add_rmsnorm_dispatch<true, 4>(x, res, w, y, M, H, eps, s)
                : add_rmsnorm_dispatch<false, 4>(x, res, w, y, M, H, eps, s);
  return bf16 ? add_rmsnorm_dispatch<true, 1>(x, res, w, y, M, H, eps, s)
              : add_rmsnorm_dispatch<false, 1>(x, res, w, y, M, H, eps, s);
}

}  // namespace opscale
