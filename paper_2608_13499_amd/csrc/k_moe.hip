// Mixture-of-experts FFN (the FusedMoE operator): top-k routing, and the
// routed expert SwiGLU MLPs with the routing-weighted sum.
//
// The expert MLPs run as two grouped GEMMs over the token-slot pairs sorted
// by expert, so each expert's weights are streamed once per tile-row of its
// tokens:
//   1. sort (stable, deterministic): counts of each expert per block of
//      entries, an exclusive scan (expert row offsets and tile offsets), then a
//      scatter in entry order (one kernel for short lists, three for long
//      ones), so pair i = t * topk + j lands at row pos[i] and row p of
//      the sorted list reads token gather[p];
//   2. gate_up[p] = W1[e] x[gather[p]]   (grouped GEMM, rows gathered);
//   3. act[p] = silu(gate_up[p, :F]) * gate_up[p, F:]   (the SwiGLU kernel);
//   4. y[p] = W2[e] act[p]               (grouped GEMM);
//   5. out[t] = sum_j w[t, j] y[pos[t * topk + j]], in slot order (fp32).
// Everything is ordered, so results are bitwise reproducible.
#include <algorithm>
#include <cmath>

#include <cstdlib>
#include <cstring>

#include "common.h"
#include "launch.h"

namespace opscale {

namespace {
constexpr int kSortChunk = 512;  // routing entries per sort block
constexpr int kMaxExperts = 1024;

__device__ __forceinline__ uint64_t lanemask_lt(int lane) { return lane ? (~0ull >> (64 - lane)) : 0ull; }

// ---------------------------------------------------------------- routing ----
// One wave per token.  Lane l holds logits l, l + 64, ...; the softmax
// denominator uses all E logits; the k largest are taken one at a time (the
// lowest expert index among equal logits first).
template <int VPL>
__global__ __launch_bounds__(256) void moe_topk_kernel(const float* __restrict__ logits, int32_t* __restrict__ ids,
                                                       float* __restrict__ wts, int64_t T, int E, int k,
                                                       int renormalize) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const float* row = logits + t * E;
  float v[VPL];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int e = lane + 64 * i;
    v[i] = e < E ? row[e] : -INFINITY;
    mx = fmaxf(mx, v[i]);
  }
  mx = wave_max_f(mx);
  float den = 0.f;
#pragma unroll
  for (int i = 0; i < VPL; ++i)
    if (lane + 64 * i < E) den += expf(v[i] - mx);
  den = wave_sum(den);
  uint32_t taken = 0;
  float my_w = 0.f, wsum = 0.f;  // lane j keeps the j-th pick
  int my_e = 0;
  for (int j = 0; j < k; ++j) {
    // this lane's best untaken (value, index)
    float bv = -INFINITY;
    int bi = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int e = lane + 64 * i;
      if (e < E && !(taken >> i & 1u) && (v[i] > bv || (v[i] == bv && e < bi))) {
        bv = v[i];
        bi = e;
      }
    }
    // the wave's best value, then the lowest index that has it: DPP reductions
    // (a shuffle is an LDS round trip, twelve of them a pick: top-8 of 64
    // experts over 256 tokens 7.9 -> 5.0 us)
    const float best = wave_max_f(bv);
    bi = -wave_max_i(bv == best ? -bi : -0x7fffffff);
    bv = best;
    if ((bi & 63) == lane) taken |= 1u << (bi >> 6);
    const float w = expf(bv - mx) / den;
    if (lane == j) {
      my_w = w;
      my_e = bi;
    }
    wsum += w;
  }
  if (lane < k) {
    ids[t * k + lane] = my_e;
    wts[t * k + lane] = renormalize ? my_w / wsum : my_w;
  }
}

// ------------------------------------------------------------------- sort ----
// Lanes of the wave with this lane's expert (ok lanes; e < 2^ebits): one ballot
// per bit of the index.  A loop over the distinct experts of the 64 entries,
// with an LDS round trip each, took the scatter of 2048 entries over 64
// experts to 80 us.
__device__ __forceinline__ uint64_t same_expert(int e, bool ok, int ebits) {
  uint64_t m = __builtin_amdgcn_ballot_w64(ok);
  for (int b = 0; b < ebits; ++b) {
    const uint64_t set = __builtin_amdgcn_ballot_w64((e >> b) & 1);
    m &= (e >> b) & 1 ? set : ~set;
  }
  return m;
}

// The whole sort in one workgroup of 16 waves, for the lists a layer's batch
// usually has: wave q takes the q-th sixteenth of the entries, counts its
// experts (LDS), the counts are scanned over waves and experts, and each wave
// then places its entries in order.  Two launches and two round trips of the
// counts through memory less than the kernels below, but one CU's loads: 5 us
// for 2048 entries of 64 experts against 14 in three kernels, 20 against 16
// for 17742 entries of 8.  The line lies between them.
constexpr int kOneWgMaxE = 256;
constexpr int64_t kOneWgMaxR = 8192;
__global__ __launch_bounds__(1024) void moe_sort_kernel(const int32_t* __restrict__ ids, int R, int E, int k, int ebits,
                                                        int tile_rows, int32_t* __restrict__ rows,
                                                        int32_t* __restrict__ tiles, int32_t* __restrict__ gather,
                                                        int32_t* __restrict__ pos) {
  constexpr int Q = 16;
  __shared__ int32_t next[Q][kOneWgMaxE];
  __shared__ int32_t wsum[2][kOneWgMaxE / 64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int per = ((R + Q - 1) / Q + 63) / 64 * 64;  // whole waves of entries
  const int begin = q * per, end = min(R, begin + per);
  for (int e = lane; e < E; e += 64) next[q][e] = 0;
  __syncthreads();
  for (int i = begin + lane; i < end; i += 64) {
    const int e = ids[i];
    if (e >= 0 && e < E) atomicAdd(&next[q][e], 1);  // integer counts: the order does not matter
  }
  __syncthreads();
  // thread e: expert e's total over the waves, scanned over the experts
  const int e = threadIdx.x;
  int tot = 0;
  if (e < E)
    for (int qq = 0; qq < Q; ++qq) tot += next[qq][e];
  const int nt = (tot + tile_rows - 1) / tile_rows;
  int sr = tot, st = nt;  // inclusive scans over the wave
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int ur = __shfl_up(sr, o, 64), ut = __shfl_up(st, o, 64);
    if (lane >= o) {
      sr += ur;
      st += ut;
    }
  }
  if (lane == 63 && q < kOneWgMaxE / 64) {
    wsum[0][q] = sr;
    wsum[1][q] = st;
  }
  __syncthreads();
  if (e < E) {
    int r0 = sr - tot, t0 = st - nt;
    for (int qq = 0; qq < q; ++qq) {
      r0 += wsum[0][qq];
      t0 += wsum[1][qq];
    }
    rows[e] = r0;
    tiles[e] = t0;
    if (e == E - 1) {
      rows[E] = r0 + tot;
      tiles[E] = t0 + nt;
    }
    for (int qq = 0; qq < Q; ++qq) {
      const int c = next[qq][e];
      next[qq][e] = r0;
      r0 += c;
    }
  }
  __syncthreads();
  // (the waves' tables are their own from here on: no further barrier, but a
  // wave's reads of a table row come before its writes to it)
  for (int base = begin; base < end; base += 64) {
    const int i = base + lane;
    const int ei = i < end ? ids[i] : -1;
    const bool ok = ei >= 0 && ei < E;
    const uint64_t same = same_expert(ei, ok, ebits);
    const uint64_t before = same & lanemask_lt(lane);
    int p = -1;
    if (ok) {
      p = next[q][ei] + __builtin_popcountll(before);
      gather[p] = i / k;
    }
    if (i < end) pos[i] = p;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (ok && !before) next[q][ei] += __builtin_popcountll(same);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// counts[b][e]: entries of block b routed to expert e (ids outside [0, E) are
// not counted).
__global__ __launch_bounds__(64) void moe_count_kernel(const int32_t* __restrict__ ids, int64_t R, int E,
                                                       int32_t* __restrict__ counts) {
  __shared__ int32_t cnt[kMaxExperts];
  for (int e = threadIdx.x; e < E; e += 64) cnt[e] = 0;
  __syncthreads();
  const int64_t begin = (int64_t)blockIdx.x * kSortChunk, end = min(R, begin + kSortChunk);
  for (int64_t i = begin + threadIdx.x; i < end; i += 64) {
    const int e = ids[i];
    if (e >= 0 && e < E) atomicAdd(&cnt[e], 1);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += 64) counts[(int64_t)blockIdx.x * E + e] = cnt[e];
}

// counts[b][e] becomes the exclusive prefix over the blocks; rows[e] / tiles[e]
// the exclusive prefixes over the experts of the totals and of their tile
// counts (tile_rows rows per tile); rows[E], tiles[E] the sums.  16 waves:
// for 64 experts at a time, wave q sums its range of blocks, wave 0 scans, and
// each wave then writes its range's running prefixes.
__global__ __launch_bounds__(1024) void moe_scan_kernel(int32_t* __restrict__ counts, int nb, int E, int tile_rows,
                                                        int32_t* __restrict__ rows, int32_t* __restrict__ tiles) {
  constexpr int Q = 16;
  __shared__ int32_t part[Q][64];
  __shared__ int32_t carry[2];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int per = (nb + Q - 1) / Q;
  const int b0 = q * per, b1 = min(nb, b0 + per);
  if (threadIdx.x == 0) carry[0] = carry[1] = 0;
  for (int e0 = 0; e0 < E; e0 += 64) {
    const int e = e0 + lane;
    int sum = 0;
    if (e < E)
      for (int b = b0; b < b1; ++b) sum += counts[(int64_t)b * E + e];
    part[q][lane] = sum;
    __syncthreads();
    if (q == 0) {
      int tot = 0;
#pragma unroll
      for (int qq = 0; qq < Q; ++qq) {
        const int c = part[qq][lane];
        part[qq][lane] = tot;  // exclusive prefix over the block ranges
        tot += c;
      }
      if (e >= E) tot = 0;
      const int nt = (tot + tile_rows - 1) / tile_rows;
      int sr = tot, st = nt;  // inclusive scans over the lanes
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int ur = __shfl_up(sr, o, 64), ut = __shfl_up(st, o, 64);
        if (lane >= o) {
          sr += ur;
          st += ut;
        }
      }
      const int cr = carry[0], ct = carry[1];
      if (e < E) {
        rows[e] = cr + sr - tot;
        tiles[e] = ct + st - nt;
      }
      const int lr = __shfl(sr, 63, 64), lt = __shfl(st, 63, 64);
      if (lane == 0) {
        carry[0] = cr + lr;
        carry[1] = ct + lt;
      }
    }
    __syncthreads();
    if (e < E) {
      int run = part[q][lane];
      for (int b = b0; b < b1; ++b) {
        const int c = counts[(int64_t)b * E + e];
        counts[(int64_t)b * E + e] = run;
        run += c;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    rows[E] = carry[0];
    tiles[E] = carry[1];
  }
}

// Entries of block b in order: entry i (token i / topk) routed to expert e
// goes to sorted row rows[e] + counts[b][e] + (its rank among block b's
// earlier entries of expert e).  pos[i] = -1 for ids outside [0, E).
__global__ __launch_bounds__(64) void moe_scatter_kernel(const int32_t* __restrict__ ids, int64_t R, int E, int k,
                                                         int ebits,
                                                         const int32_t* __restrict__ counts,
                                                         const int32_t* __restrict__ rows,
                                                         int32_t* __restrict__ gather, int32_t* __restrict__ pos) {
  __shared__ int32_t next[kMaxExperts];
  const int lane = threadIdx.x;
  for (int e = lane; e < E; e += 64) next[e] = rows[e] + counts[(int64_t)blockIdx.x * E + e];
  __syncthreads();
  const int64_t begin = (int64_t)blockIdx.x * kSortChunk, end = min(R, begin + kSortChunk);
  for (int64_t base = begin; base < end; base += 64) {
    const int64_t i = base + lane;
    const bool valid = i < end;
    const int e = valid ? ids[i] : -1;
    const bool ok = valid && e >= 0 && e < E;
    if (valid && !ok) pos[i] = -1;
    const uint64_t same = same_expert(e, ok, ebits);
    if (ok) {
      const int p = next[e] + __builtin_popcountll(same & lanemask_lt(lane));
      gather[p] = (int32_t)(i / k);
      pos[i] = p;
    }
    __syncthreads();  // every lane has read next[e] (one wave: a wait, not a barrier)
    if (ok && !(same & lanemask_lt(lane))) next[e] += __builtin_popcountll(same);
    __syncthreads();
  }
}

// ---------------------------------------------------------------- combine ----
// out[t] = sum_j w[t, j] y[pos[t * k + j]] (slots in order, fp32): 8 columns per
// thread, 2048 per workgroup (grid.y covers H; one workgroup a token, each
// thread with two dependent rounds of loads, took 256 tokens of top-8 10.9
// instead of 7.2 us).  The rows of kBatch slots are requested together.
__global__ __launch_bounds__(256) void moe_combine_kernel(const __bf16* __restrict__ y, const int32_t* __restrict__ pos,
                                                          const float* __restrict__ wts, __bf16* __restrict__ out,
                                                          int H, int k) {
  constexpr int kBatch = 8;
  const int64_t t = blockIdx.x;
  const int c = ((int)blockIdx.y * 256 + (int)threadIdx.x) * 8;
  if (c < H) {
    float acc[8] = {};
    for (int j0 = 0; j0 < k; j0 += kBatch) {
      u32x4 v[kBatch];
      int p[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) p[j] = j0 + j < k ? pos[t * k + j0 + j] : -1;
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
        if (p[j] >= 0) v[j] = *reinterpret_cast<const u32x4*>(y + (int64_t)p[j] * H + c);
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        if (p[j] < 0) continue;
        const float w = wts[t * k + j0 + j];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[2 * q] += w * bf_lo(v[j][q]);
          acc[2 * q + 1] += w * bf_hi(v[j][q]);
        }
      }
    }
    *reinterpret_cast<u32x4*>(out + t * H + c) =
        u32x4{pack_bf2(acc[0], acc[1]), pack_bf2(acc[2], acc[3]), pack_bf2(acc[4], acc[5]), pack_bf2(acc[6], acc[7])};
  }
}

inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

struct MoeWorkspace {
  int32_t *counts, *rows, *tiles, *gather, *pos;
  __bf16 *gate_up, *act, *y;
  size_t bytes;
};

MoeWorkspace carve(void* base, int64_t T, int H, int F, int E, int k) {
  const int64_t R = T * k;
  const int64_t nb = (R + kSortChunk - 1) / kSortChunk;
  MoeWorkspace w{};
  char* p = static_cast<char*>(base);
  size_t off = 0;
  auto take = [&](size_t b) {
    char* q = p ? p + off : nullptr;
    off += align256(b);
    return q;
  };
  w.counts = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)std::max<int64_t>(1, nb) * E));
  w.rows = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)(E + 1)));
  w.tiles = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)(E + 1)));
  w.gather = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)R));
  w.pos = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)R));
  w.gate_up = reinterpret_cast<__bf16*>(take(2 * (size_t)R * 2 * F));
  w.act = reinterpret_cast<__bf16*>(take(2 * (size_t)R * F));
  w.y = reinterpret_cast<__bf16*>(take(2 * (size_t)R * H));
  w.bytes = off;
  return w;
}
}  // namespace

int32_t moe_max_experts() { return kMaxExperts; }

size_t moe_workspace_bytes(int64_t T, int32_t H, int32_t F, int32_t E, int32_t topk) {
  return carve(nullptr, T, H, F, E, topk).bytes;
}

hipError_t launch_moe_topk(const float* logits, int32_t* ids, float* wts, int64_t T, int32_t E, int32_t k,
                           bool renormalize, hipStream_t s) {
  const dim3 grid((unsigned)((T + 3) / 4)), block(256);
  const int vpl = (E + 63) / 64;
#define OPS_TOPK(V) \
  hipLaunchKernelGGL((moe_topk_kernel<V>), grid, block, 0, s, logits, ids, wts, T, E, k, (int)renormalize)
  if (vpl <= 1) OPS_TOPK(1);
  else if (vpl <= 2) OPS_TOPK(2);
  else if (vpl <= 4) OPS_TOPK(4);
  else if (vpl <= 8) OPS_TOPK(8);
  else OPS_TOPK(16);
#undef OPS_TOPK
  return hipGetLastError();
}

hipError_t launch_fused_moe(const void* x, const void* w1, const void* w2, const int32_t* ids, const float* wts,
                            void* out, int64_t T, int32_t H, int32_t F, int32_t E, int32_t k, void* ws,
                            hipStream_t s) {
  const int64_t R = T * k;
  const int nb = (int)((R + kSortChunk - 1) / kSortChunk);
  const MoeWorkspace w = carve(ws, T, H, F, E, k);
  const int32_t bm = grouped_gemm_tile_rows(R, E);
  int ebits = 0;
  while ((1 << ebits) < E) ++ebits;
  hipError_t e;
  if (E <= kOneWgMaxE && R <= kOneWgMaxR) {
    hipLaunchKernelGGL(moe_sort_kernel, dim3(1), dim3(1024), 0, s, ids, (int)R, E, k, ebits, bm, w.rows, w.tiles,
                       w.gather, w.pos);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  } else {
    hipLaunchKernelGGL(moe_count_kernel, dim3((unsigned)nb), dim3(64), 0, s, ids, R, E, w.counts);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(moe_scan_kernel, dim3(1), dim3(1024), 0, s, w.counts, nb, E, bm, w.rows, w.tiles);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(moe_scatter_kernel, dim3((unsigned)nb), dim3(64), 0, s, ids, R, E, k, ebits, w.counts, w.rows,
                       w.gather, w.pos);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // act = silu(W1g[e] x[token]) * (W1u[e] x[token])   (rows gathered), [R, F]:
  // the SwiGLU sits in the GEMM's epilogue when an expert's gate-up weight
  // spans less than 4 GB (32-bit row offsets); else gate_up [R, 2F] first
  // (OPSCALE_TUNE_MOE_FUSE = 0 forces the unfused path, for tests)
  if ((int64_t)2 * F * H * 2 < ((int64_t)1 << 32) && tuning(OPSCALE_TUNE_MOE_FUSE) != 0) {
    if ((e = launch_gemm_grouped(x, T, w1, (int64_t)2 * F * H, w.act, R, 2 * (int64_t)F, H, E, bm, w.gather, w.rows,
                                 w.tiles, F, s)) != hipSuccess)
      return e;
  } else {
    if ((e = launch_gemm_grouped(x, T, w1, (int64_t)2 * F * H, w.gate_up, R, 2 * (int64_t)F, H, E, bm, w.gather,
                                 w.rows, w.tiles, 0, s)) != hipSuccess)
      return e;
    if ((e = launch_swiglu(w.gate_up, w.act, R, F, true, s)) != hipSuccess) return e;
  }
  // y = W2[e] act   (sorted rows), [R, H]
  if ((e = launch_gemm_grouped(w.act, R, w2, (int64_t)H * F, w.y, R, H, F, E, bm, nullptr, w.rows, w.tiles, 0, s)) !=
      hipSuccess)
    return e;
  hipLaunchKernelGGL(moe_combine_kernel, dim3((unsigned)T, (unsigned)((H + 2047) / 2048)), dim3(256), 0, s, w.y, w.pos, wts,
                     static_cast<__bf16*>(out), H, k);
  return hipGetLastError();
}

}  // namespace opscale
