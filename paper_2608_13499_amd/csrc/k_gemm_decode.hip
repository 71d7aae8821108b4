// Linear layers at decode-batch M (up to 128 rows): y[M,N] = x[M,K] W[N,K]^T.
//
// Every weight byte is read once from HBM and used for only M flops: the
// weight stream bounds these, and everything else has to stay out of its way.
//
// A workgroup of NW waves owns 16 NW output columns and all M rows over one K
// range, in slices of 64 k:
//  * each wave streams its own 16 weight rows straight into registers, seven
//    slices ahead of the one in use (a ring of eight); no LDS on this path;
//  * the x slice of all M rows is shared through a 4-stage LDS ring filled by
//    LDS DMA (x is small and stays in L2: every workgroup reads it);
//  * MFMA 16x16x32 with the weight fragment as A and the x fragment as B, so a
//    lane's accumulator holds one x row and four consecutive output columns.
//
// Two things decide the rate (us; gate-up 28672 x 4096, M = 48: 54.7 before
// either, floor 36.6 at 6.5 TB/s):
//  * NW is 5 to 8, whichever gives workgroups and K ranges that fill whole
//    rounds of the CUs with the fewest bytes each: a CU's loads alone cannot
//    make up for idle ones (28672 columns as 224 workgroups of 128: 51.8, as
//    256 of 112 columns: 49);
//  * each workgroup starts its K range at another slice and wraps around.  In
//    step along K, all of them would read the same few k of rows a power of
//    two apart, i.e. the same few HBM channels: 49 -> 42.2 (57344 x 8192: 191 ->
//    169).  A ring of 16 slices changes nothing, nontemporal loads cost 1-10 %.
//
// K is split over workgroups when the columns alone give fewer than about one
// workgroup per CU; the fp32 partials go to the caller's workspace and are
// summed in split order by a second kernel (deterministic).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gemm_schedule.h"
#include "launch.h"

namespace opscale {

namespace {

constexpr int kBK = 64;       // K per slice
constexpr int kSlots = 8;     // weight ring (registers)
constexpr int kAhead = 7;     // weight slices in flight beyond the one in use
constexpr int kStages = 4;    // x ring (LDS)
static_assert(kAhead == kSlots - 1 && kSlots % kStages == 0, "ring shapes");

template <int V>
using Int = std::integral_constant<int, V>;

// f(Int<0>), ..., f(Int<N - 1>)
template <int N, class F, int I = 0>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(Int<I>{});
    static_for<N, F, I + 1>(static_cast<F&&>(f));
  }
}

}  // namespace

// M <= 16 * TM.  Grid: tiles_n x nsplit workgroups of NW waves.
// x and W are deliberately not __restrict__: with it the compiler treats
// their loads as invariant and moves them across the fences below.
template <int TM, int NW>
__global__ __launch_bounds__(64 * NW, 1) void gemm_decode_bf16_kernel(const __bf16* x, const __bf16* W,
                                                                      const __bf16* __restrict__ bias,
                                                                      __bf16* __restrict__ y, int M, int N, int K,
                                                                      int kchunk, int tiles_n,
                                                                      float* __restrict__ part) {
  // one x slice: 2 TM loads of 1 KB (8 rows each) over the waves; every wave
  // issues XL of them (those past the rows read zeros), so the wait below is
  // one constant
  constexpr int XL = (2 * TM + NW - 1) / NW;
  constexpr int kStageBytes = XL * NW * 1024;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  OPS_LDS char* smem = (OPS_LDS char*)smem_raw;

  // Consecutive ids on one XCD (so one XCD mostly reads one K range of x),
  // split-major.
  const uint32_t id = xcd_remap(blockIdx.x, gridDim.x);
  const int split = (int)(id / (uint32_t)tiles_n), tn = (int)(id % (uint32_t)tiles_n);
  const int k0 = split * kchunk;
  const int Kr = min(K - k0, kchunk);
  const int ns = Kr / kBK;
  // the slice this workgroup starts at (the column tiles spread over K)
  const int rot = tiles_n <= 65536 ? (int)((uint32_t)(tn * ns) / (uint32_t)tiles_n) : tn % ns;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int fr = lane & 15, fq = lane >> 4;
  const int n0 = (tn * NW + wave) * 16;  // this wave's first weight row (output column)
  const int wrows = max(0, min(16, N - n0));
  // rows past N and past M read as zeros (buffer range check)
  const __bf16* wp = W + (int64_t)min(n0, N - 1) * K + k0;
  const uint32_t wrec = wrows > 0 ? (uint32_t)(((int64_t)(wrows - 1) * K + Kr) * 2) : 0u;
  const __bf16* xp = x + k0;
  const uint32_t xrec = (uint32_t)(((int64_t)(M - 1) * K + Kr) * 2);
  const uint32_t w_voff = (uint32_t)((fr * K + 8 * fq) * 2);

  // x DMA: load g of this wave covers rows 8 (g NW + wave) .. + 7; lane p
  // writes physical chunk p % 8 of row p / 8 of them (chunk c of row r at
  // c ^ (r mod 8): the fragment reads are free of bank conflicts).
  uint32_t x_voff[XL];
#pragma unroll
  for (int g = 0; g < XL; ++g) {
    const int r = (g * NW + wave) * 8 + lane / 8;
    x_voff[g] = r < M ? (uint32_t)((r * K + (((lane & 7) ^ (r & 7)) << 3)) * 2) : kOobOffset;
  }
  // fragment of k-step j: row fr of each 16-row block, chunk 4 j + fq
  int frag_off[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) frag_off[j] = fr * 128 + (((4 * j + fq) ^ (fr & 7)) << 4);

  bf16x8 wf[kSlots][2];
  f32x4 acc[TM];
#pragma unroll
  for (int t = 0; t < TM; ++t) acc[t] = f32x4{};

  // Slice s of the range, in this workgroup's order.  Loads past the last one
  // are issued too, on a descriptor of no records (zeros into a stage or slot
  // no step reads any more): every step then issues the same loads.
  auto slice = [&](int s) { return s + rot < ns ? s + rot : s + rot - ns; };
  auto load_x = [&](int s, int stage) {
    const __amdgpu_buffer_rsrc_t r = make_rsrc(xp + (int64_t)slice(s) * kBK, s < ns ? xrec : 0u);
#pragma unroll
    for (int g = 0; g < XL; ++g)
      buffer_load16_lds<kNoL1>(r, smem + stage * kStageBytes + (g * NW + wave) * 1024, x_voff[g]);
  };
  auto load_w = [&](auto slot_c, int s) {
    constexpr int slot = decltype(slot_c)::value;
    const __amdgpu_buffer_rsrc_t r = make_rsrc(wp + (int64_t)slice(s) * kBK, s < ns ? wrec : 0u);
#pragma unroll
    for (int j = 0; j < 2; ++j) wf[slot][j] = __builtin_bit_cast(bf16x8, buffer_load16(r, w_voff + 64 * j));
  };
  // The counted wait holds only in the issue order below, which fence() fixes:
  // the compiler would otherwise move weight loads in between the DMA loads.
  auto fence = [] { asm volatile("" ::: "memory"); };

  // Step c (slot c % kSlots, stage c % kStages): wait for x slice c, barrier
  // (every wave is done with the stage of slice c - 1), refill that stage and
  // the slot of slice c - 1, then the slice's fragment reads and MFMAs.
  auto step = [&](auto slot_c, int c) {
    constexpr int slot = decltype(slot_c)::value;
    constexpr int stage = slot % kStages;
    // newer than X(c): the W loads of its own step, X and W of the two since
    wait_vmcnt_le<2 * (kStages - 1) + XL * (kStages - 2)>();
    barrier_keep_loads();
    load_x(c + kStages - 1, (stage + kStages - 1) % kStages);
    fence();
    load_w(Int<(slot + kAhead) % kSlots>{}, c + kAhead);
    fence();
    bf16x8 xf[2][TM];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < TM; ++t)
        xf[j][t] = *reinterpret_cast<const OPS_LDS bf16x8*>(smem + stage * kStageBytes + frag_off[j] + t * 2048);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < TM; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[slot][j], xf[j][t], acc[t], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

  // Prologue: the loads steps -kAhead .. -1 would have issued, in their order.
  static_for<kAhead>([&](auto i_c) {
    constexpr int i = decltype(i_c)::value, xs = i - kAhead + kStages - 1;
    if constexpr (xs >= 0) {
      load_x(xs, xs % kStages);
      fence();
    }
    load_w(Int<i>{}, i);
    fence();
  });
  // Whole rounds of kSlots steps, every step unconditional: slices past the
  // last read as zeros, so a partial last round only adds MFMAs on zeros.
  // Every load is then issued exactly as written (a weight load that only a
  // conditional later step used was sunk by the compiler into that step, past
  // the barriers the wait counts rely on).
  for (int base = 0; base < ns; base += kSlots)
    static_for<kSlots>([&](auto s_c) { step(s_c, base + decltype(s_c)::value); });
  wait_vmem();  // no LDS DMA may still be in flight when the workgroup ends

  // Lane (fr, fq) of block t holds x row 16 t + fr, columns n0 + 4 fq .. + 3.
  const int n = n0 + 4 * fq;
  if (n >= N) return;
  if (part) {
    float* pbase = part + (int64_t)split * M * N;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int m = 16 * t + fr;
      if (m < M) *reinterpret_cast<f32x4*>(pbase + (int64_t)m * N + n) = acc[t];
    }
    return;
  }
  float b[4] = {};
  if (bias) {
    const u32x2 bb = *reinterpret_cast<const u32x2*>(bias + n);
    b[0] = bf_lo(bb[0]);
    b[1] = bf_hi(bb[0]);
    b[2] = bf_lo(bb[1]);
    b[3] = bf_hi(bb[1]);
  }
#pragma unroll
  for (int t = 0; t < TM; ++t) {
    const int m = 16 * t + fr;
    if (m < M)
      *reinterpret_cast<u32x2*>(y + (int64_t)m * N + n) =
          u32x2{pack_bf2(acc[t][0] + b[0], acc[t][1] + b[1]), pack_bf2(acc[t][2] + b[2], acc[t][3] + b[3])};
  }
}

bool decode_linear_supported(int64_t M, int64_t N, int64_t K) {
  // (four threads a column: a grid holds fewer than 2^32)
  return M >= 1 && M <= kDecodeMaxM && K % kBK == 0 && N >= 1 && N < ((int64_t)1 << 30) && K <= (1 << 20);
}

namespace {
struct DecodeShape {
  int waves;      // 16 columns each
  int splits;     // K ranges
  int64_t chunk;  // slices per range
};

// The waves per workgroup (and K ranges of at least 8 slices, at most about
// one workgroup per CU in all) with the fewest weight bytes per CU: rounds x
// columns x slices, slices in whole rounds of the weight ring.
DecodeShape decode_shape(int64_t N, int64_t K) {
  const int64_t ns = K / kBK;
  DecodeShape best{};
  int64_t best_cost = 0;
  for (int nw = kMaxStreamWaves; nw >= kMinStreamWaves; --nw) {
    const int64_t tiles = (N + 16 * nw - 1) / (16 * nw);
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(kNumCUs / tiles, ns / 8));
    const int64_t chunk = (ns + most - 1) / most, splits = (ns + chunk - 1) / chunk;
    const int64_t rounds = (tiles * splits + kNumCUs - 1) / kNumCUs;
    const int64_t cost = rounds * nw * ((chunk + kSlots - 1) / kSlots);
    if (best_cost == 0 || cost < best_cost) {
      best_cost = cost;
      best = {nw, (int)splits, chunk};
    }
  }
  return best;
}
}  // namespace

int decode_linear_splits(int64_t M, int64_t N, int64_t K) {
  (void)M;
  return decode_shape(N, K).splits;
}

size_t decode_linear_ws_bytes(int64_t M, int64_t N, int64_t K) {
  const int s = decode_linear_splits(M, N, K);
  return s > 1 ? (size_t)s * M * N * sizeof(float) : 0;
}

template <int TM, int NW>
static hipError_t launch_decode(const void* x, const void* W, const void* bias, void* y, int64_t M, int64_t N,
                                int64_t K, int nsplit, int64_t chunk, float* part, hipStream_t s) {
  constexpr int lds = kStages * ((2 * TM + NW - 1) / NW) * NW * 1024;
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(gemm_decode_bf16_kernel<TM, NW>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr != hipSuccess) return attr;
  const int64_t tiles = (N + 16 * NW - 1) / (16 * NW);
  hipLaunchKernelGGL((gemm_decode_bf16_kernel<TM, NW>), dim3((unsigned)(tiles * nsplit)), dim3(64 * NW), lds, s,
                     static_cast<const __bf16*>(x), static_cast<const __bf16*>(W), static_cast<const __bf16*>(bias),
                     static_cast<__bf16*>(y), (int)M, (int)N, (int)K, (int)(chunk * kBK), (int)tiles,
                     nsplit > 1 ? part : nullptr);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || nsplit <= 1) return e;
  return launch_splitk_reduce(part, nsplit, bias, y, M, N, s);
}

// splits <= 1: one K range; otherwise the ranges decode_linear_splits counts.
hipError_t launch_linear_decode(const void* x, const void* W, const void* bias, void* y, int64_t M, int64_t N,
                                int64_t K, int splits, void* ws, hipStream_t s) {
  const DecodeShape sh = decode_shape(N, K);
  const int nsplit = splits > 1 ? sh.splits : 1;
  const int64_t chunk = splits > 1 ? sh.chunk : K / kBK;
  // (the K ranges are fixed with the workspace, the columns of a workgroup are not)
  const int cus = stream_cus(s);
  const int waves = cus < kNumCUs ? stream_waves(N, nsplit, cus) : sh.waves;
  const auto rows = [&](auto tm_c) {
    constexpr int TM = decltype(tm_c)::value;
    float* part = static_cast<float*>(ws);
    switch (waves) {
      case 5: return launch_decode<TM, 5>(x, W, bias, y, M, N, K, nsplit, chunk, part, s);
      case 6: return launch_decode<TM, 6>(x, W, bias, y, M, N, K, nsplit, chunk, part, s);
      case 7: return launch_decode<TM, 7>(x, W, bias, y, M, N, K, nsplit, chunk, part, s);
      default: return launch_decode<TM, 8>(x, W, bias, y, M, N, K, nsplit, chunk, part, s);
    }
  };
  if (M <= 16) return rows(Int<1>{});
  if (M <= 32) return rows(Int<2>{});
  if (M <= 64) return rows(Int<4>{});
  return rows(Int<8>{});
}

}  // namespace opscale
