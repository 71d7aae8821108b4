// Linear layers y[M,N] = x[M,K] W[N,K]^T (+ bias): QKV, O, gate-up and down
// projections of the decoder layer.
//
// bf16 path: MFMA v_mfma_f32_16x16x32_bf16, fp32 accumulation.  A 256x256
// block tile is staged through an LDS ring in BK-wide K slices; the next slices
// are fetched with buffer_load ... lds (HBM/L2 -> LDS without passing through
// registers) while the current one feeds the matrix cores.  Large problems
// use four waves of 128x128 sub-tiles, one per SIMD, with the accumulators in
// AGPRs (gemm_bf16_w4_kernel), the grouped mixture-of-experts GEMMs among them;
// the eight-wave form of the same tile (two waves of 128x64 per SIMD) takes
// what that kernel's chains and 32-bit offsets do not.  Sizes that give few such
// tiles take 128x256 ones (gemm_bf16_h4_kernel) where that is faster, and
// decode-sized M splits K.  (192x256 and 256x128 tiles, CfgT192 and CfgMid, run
// only where the tile knob asks for them.)  Rows and K columns beyond the matrix
// read as zeros through the buffer descriptor's range check, so ragged M, N and
// K need no separate code path.
//
// Both operands are K-contiguous, which is what an MFMA operand lane wants: a
// lane holds 8 consecutive k of one row.  The W tile is the MFMA "A" operand
// and the x tile the "B" operand, so each accumulator lane owns one output row
// m and runs of 4 consecutive columns n, stored as 8-byte chunks.
//
// (fp32: k_gemm_f32.hip.)
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "gemm_schedule.h"
#include "common.h"
#include "launch.h"

namespace opscale {

namespace {

constexpr int64_t kGroupBytes = (int64_t)16 << 20;  // x rows per tile group (see tile_group_rows)
constexpr int64_t kW4MaxN = (int64_t)1 << 22;  // the four-wave kernel's 32-bit offsets into 256 rows of y
constexpr int64_t kSplitKMaxM = 2048;  // split-K is for small M (decode batches)

// Tile configuration: BM x BN block tile, K in slices of BK, WGM x WGN waves
// (each owns a (BM/WGM) x (BN/WGN) sub-tile), STAGES-deep LDS ring.
// DEEP: the ring keeps STAGES - 1 slices in flight while a slice is used
// (decode-sized M, where the loop waits on memory, not on the matrix cores);
// otherwise the next slice is made visible one step early so its first
// fragment reads overlap the current slice's last MFMAs.
template <int BM_, int BN_, int BK_, int WGM_, int WGN_, int STAGES_, bool DEEP_ = false>
struct GemmCfg {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_, STAGES = STAGES_;
  static constexpr bool DEEP = DEEP_;
  static constexpr int WM = BM / WGM, WN = BN / WGN;  // wave tile (m x n)
  static constexpr int kThreads = WGM * WGN * 64;
  static constexpr int kWaves = WGM * WGN;
  static constexpr int kRowBytes = BK * 2;              // one LDS row = BK bf16
  static constexpr int kCPR = BK / 8;                   // 16-byte chunks per row
  static constexpr int kRowsPerLoad = 64 / kCPR;        // rows one 1 KB wave load covers
  static constexpr int kStageBytes = (BM + BN) * kRowBytes;
  static constexpr int kLdsBytes = STAGES * kStageBytes;
  static constexpr int kLoadsPerTile = (BM + BN) / kRowsPerLoad / kWaves;  // per wave
  static_assert(BM % (kRowsPerLoad * kWaves) == 0 && BN % (kRowsPerLoad * kWaves) == 0,
                "each operand's rows must split evenly over the waves");
  // The fragment double buffer alternates by k-step within a slice and
  // restarts at buffer 0 in the next, so a slice must hold an even number of
  // 32-wide k-steps; the LDS swizzle assumes 128-byte rows.
  static_assert(BK == 64, "64-wide K slices: two 32-wide k-steps of 128-byte rows");
  static_assert(kLoadsPerTile * (STAGES - 2 > 0 ? STAGES - 2 : 0) <= 63, "vmcnt range");
};

using CfgBig8 = GemmCfg<256, 256, 64, 2, 4, 2>;    // 8 waves of 128x64, 2 x 64 KB stages
using CfgT192 = GemmCfg<192, 256, 64, 2, 4, 2>;    // 8 waves of 96x64, 2 x 56 KB stages
using CfgMid = GemmCfg<256, 128, 64, 2, 2, 3>;     // 4 waves of 128x64, 3 x 48 KB stages
using CfgW4 = GemmCfg<256, 256, 64, 2, 2, 2>;      // 4 waves of 128x128, 2 x 64 KB stages
using CfgRow64 = GemmCfg<64, 256, 64, 1, 4, 2>;    // 4 waves of 64x64, 2 x 40 KB stages (few rows)
// split-K tiles for decode-sized M: a K range is short, so the ring is deep
using CfgSk64 = GemmCfg<64, 256, 64, 1, 4, 4, true>;    // M <= 64: 4 waves of 64x64, 4 x 40 KB stages
using CfgSk128 = GemmCfg<128, 256, 64, 2, 4, 3, true>;  // 65 to 128 rows: 8 waves of 64x64, 3 x 48 KB stages


// 16-byte chunk c of LDS row r is stored at physical chunk c ^ swz(r).
// gfx950 LDS has 64 banks of 4 bytes and serves a 16-byte-per-lane read in
// four passes of 16 lanes: pass 2 * (lane / 32) + parity of bits 2..4 of the
// lane (lanes in 4-lane blocks, blocks of odd and even bit parity alternating;
// measured).  A 16x16x32 operand read puts row lane % 16 and logical chunk
// 4 ks + lane / 16 in each lane, so a pass holds 8 rows of one parity class at
// each of two chunks; XOR with the row mod 8 gives those 16 lanes 16
// distinct 16-byte bank groups for both k-steps of a 64-wide slice.  swz depends only
// on the row mod 16, i.e. on the lane, so one per-lane offset per K step
// serves every 16-row fragment of a wave (the rest is an immediate offset).
template <int CPR>
__device__ __forceinline__ int swz(int r) {
  static_assert(CPR == 8, "128-byte rows");
  return r & 7;
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding:
// vmcnt in bits [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// One BK-wide slice of ROWS rows of a K-contiguous bf16 matrix (descriptor
// based at the tile's first row) into an LDS stage region.  Wave w issues
// loads w, w + waves, ...; lane p of a load writes LDS bytes [p*16, p*16+16)
// of its 1 KB group: row p / CPR, physical chunk p % CPR.
// A row that must read as zeros (past the end of a grouped operand).
constexpr uint32_t kNoRow = 0xffffffffu;

// row_off[g]: byte offset of the row this lane loads in its g-th load group
// (kNoRow: a row that reads as zeros).
template <class C, int ROWS>
__device__ __forceinline__ void load_slice(__amdgpu_buffer_rsrc_t rsrc, OPS_LDS char* lds, const uint32_t* row_off,
                                           int K, int k0, int wave, int lane) {
  const int rl = lane / C::kCPR, pc = lane % C::kCPR;
  constexpr int kPerWave = ROWS / C::kRowsPerLoad / C::kWaves;
#pragma unroll
  for (int g = 0; g < kPerWave; ++g) {
    const int grp = g * C::kWaves + wave;
    const int r = grp * C::kRowsPerLoad + rl;
    const int c = pc ^ swz<C::kCPR>(r);
    const int k = k0 + c * 8;
    const uint32_t voff = (k < K && row_off[g] != kNoRow) ? row_off[g] + (uint32_t)k * 2u : kOobOffset;
    buffer_load16_lds<kNoL1>(rsrc, lds + grp * 1024, voff);
  }
}

template <class C>
__device__ __forceinline__ bf16x8 lds_frag(const OPS_LDS char* p) {
  return *reinterpret_cast<const OPS_LDS bf16x8*>(p);
}

}  // namespace

// Tile (tm, tn) of plain-GEMM tile id tid in grouped order: group_m
// tile-rows sweep the tile-columns together, so a W column-block is fetched
// once per group and reused from L2 / MALL by every tile-row of the group
// while the group's x rows stay cache resident.
__device__ __forceinline__ void tile_coords(uint32_t tid, int tiles_m, int tiles_n, int group_m, int& tm, int& tn) {
  const int group = tid / (group_m * tiles_n);
  const int first_m = group * group_m;
  const int gsize = min(tiles_m - first_m, group_m);
  const int in_group = tid % (group_m * tiles_n);
  tm = first_m + in_group % gsize;
  tn = in_group / gsize;
}

// Split-K (splits > 1): workgroup blockIdx.x / tiles takes the K range
// [split * kchunk, (split + 1) * kchunk) and writes its fp32 partial tile to
// part[split][M][N] (no bias); a second kernel sums the splits in order.
//
// Split tail (tail_cnt > 0): workgroups [0, dp_cnt) take whole tiles 0 ..
// dp_cnt - 1 (full K, results to y); the rest take the K ranges of the last
// tail_cnt tiles: item b (from dp_cnt) covers tile dp_cnt + b % tail_cnt, K
// range b / tail_cnt, and writes its fp32 tile compactly to
// part[(split * tail_cnt + tile - dp_cnt) * BM * BN] (row-major BM x BN); a
// second kernel sums those in split order.  Runs a launch whose last round
// would be mostly idle at a fraction of a tile's time.
//
// GROUPED (one GEMM per expert of a mixture-of-experts layer): the output
// rows are grouped by expert, expert e owning rows [rows[e], rows[e + 1]) in
// tiles tiles[e] .. tiles[e + 1] - 1 of BM rows; workgroup (tile t, column
// block n) multiplies by W + e * w_stride, and output row m reads x row
// gather[m] (m itself when gather is null).  x then has x_rows rows.
struct GroupedGemm {
  const int32_t* gather;  // output row -> x row (null: the identity)
  const int32_t* rows;    // [E + 1]
  const int32_t* tiles;   // [E + 1]
  int E;
  int x_rows;
  int64_t w_stride;       // elements from one expert's W to the next
  // > 0: W is a gate-up projection [2F, K] (gate rows first) and y the SwiGLU
  // activation [rows, F]: output column c of the GEMM is gate row c / 2 (even
  // c) or up row F + c / 2 (odd c), so each lane's runs of 4 columns hold two
  // (gate, up) pairs and the epilogue stores silu(gate) * up.  N = 2F.
  int swiglu_f;
};

template <class C, bool GROUPED = false>
__global__ __launch_bounds__(C::kThreads, 1) void gemm_bf16_kernel(const __bf16* __restrict__ x,
                                                                   const __bf16* __restrict__ W,
                                                                   const __bf16* __restrict__ bias,
                                                                   __bf16* __restrict__ y, int M, int N,
                                                                   int K_total, int group_m, int kchunk,
                                                                   float* __restrict__ part, GroupedGemm gg,
                                                                   int dp_cnt, int tail_cnt) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  OPS_LDS char* smem = (OPS_LDS char*)smem_raw;
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, WM = C::WM, WN = C::WN, S = C::STAGES;
  // 16x16x32 MFMAs: half the length of a 32x32x16 one for the same work per
  // k-window, so the next fragments' LDS reads and the loads find twice the
  // issue slots between them (measured 0-2 % faster on every shape here)
  constexpr int MI = 16;
  constexpr int TM = WM / MI, TN = WN / MI;  // MFMA tiles per wave

  const int tiles_n = (N + BN - 1) / BN;
  const int ld = K_total;
  int m0, n0, m_rows, split = 0;
  int kc = kchunk;                  // K elements per split
  float* tile_part = nullptr;       // split tail: this item's compact partial tile
  if constexpr (GROUPED) {
    // Work items in order expert, column block, tile-row of the expert, so
    // an expert's tile-rows use one W column block back to back; spread over
    // the XCDs in contiguous ranges of the items that exist (the grid is an
    // upper bound; the workgroups past it return).
    const int total = gg.tiles[gg.E] * tiles_n;
    if ((int)blockIdx.x >= total) return;
    const int id = (int)xcd_remap(blockIdx.x, (uint32_t)total);
    int lo = 0, hi = gg.E;  // gg.tiles[lo] * tiles_n <= id < gg.tiles[hi] * tiles_n
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (gg.tiles[mid] * tiles_n <= id) lo = mid;
      else hi = mid;
    }
    const int tr_e = gg.tiles[lo + 1] - gg.tiles[lo];  // tile-rows of expert lo (>= 1)
    const int local = id - gg.tiles[lo] * tiles_n;
    const int tn = local / tr_e, tr = local - tn * tr_e;
    n0 = tn * BN;
    m0 = gg.rows[lo] + tr * BM;
    m_rows = min(BM, gg.rows[lo + 1] - m0);
    W += lo * gg.w_stride;
  } else {
    const int tiles_m = (M + BM - 1) / BM;
    const int tiles = tiles_m * tiles_n;
    uint32_t tid;
    if (tail_cnt == 0) {
      split = blockIdx.x / tiles;
      tid = xcd_remap(blockIdx.x - split * tiles, (uint32_t)tiles);
    } else if ((int)blockIdx.x < dp_cnt) {
      tid = xcd_remap(blockIdx.x, (uint32_t)dp_cnt);
      kc = K_total;
    } else {
      const int b = blockIdx.x - dp_cnt;
      split = b / tail_cnt;
      const int t = (int)xcd_remap(b - split * tail_cnt, (uint32_t)tail_cnt);
      tid = dp_cnt + t;
      tile_part = part + ((int64_t)split * tail_cnt + t) * BM * BN;
    }
    int tm, tn;
    tile_coords(tid, tiles_m, tiles_n, group_m, tm, tn);
    m0 = tm * BM;
    n0 = tn * BN;
    m_rows = min(BM, M - m0);
  }
  // this workgroup's K range: K elements starting at k_begin, rows ld apart
  const int k_begin = split * kc;
  const int K = min(K_total - k_begin, kc);

  // wave index as a scalar: the LDS destinations of the loads are then
  // wave-uniform without a readfirstlane per load
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave % C::WGM, wn = wave / C::WGM;

  // x: the tile's rows (grouped: the gathered rows of the whole operand)
  const __amdgpu_buffer_rsrc_t xr =
      GROUPED ? make_rsrc(x + k_begin, (uint32_t)(((int64_t)gg.x_rows - 1) * ld * 2 + (int64_t)K * 2))
              : make_rsrc(x + (int64_t)m0 * ld + k_begin, (uint32_t)(((int64_t)(m_rows - 1) * ld + K) * 2));
  // W: the tile's rows (fused SwiGLU: the expert's whole gate-up weight)
  const bool fused = GROUPED && gg.swiglu_f > 0;
  const __amdgpu_buffer_rsrc_t wr =
      fused ? make_rsrc(W + k_begin, (uint32_t)(((int64_t)N - 1) * ld * 2 + (int64_t)K * 2))
            : make_rsrc(W + (int64_t)n0 * ld + k_begin, (uint32_t)(((int64_t)(min(BN, N - n0) - 1) * ld + K) * 2));
  // byte offsets of the rows this lane loads (per load group)
  constexpr int LX = BM / C::kRowsPerLoad / C::kWaves, LW = BN / C::kRowsPerLoad / C::kWaves;
  uint32_t xro[LX], wro[LW];
#pragma unroll
  for (int g = 0; g < LX; ++g) {
    const int r = (g * C::kWaves + wave) * C::kRowsPerLoad + lane / C::kCPR;
    if constexpr (GROUPED) {
      const int src = r < m_rows ? (gg.gather ? gg.gather[m0 + r] : m0 + r) : -1;
      xro[g] = src >= 0 ? (uint32_t)((int64_t)src * ld * 2) : kNoRow;
    } else {
      xro[g] = (uint32_t)((int64_t)r * ld * 2);
    }
  }
#pragma unroll
  for (int g = 0; g < LW; ++g) {
    const int r = (g * C::kWaves + wave) * C::kRowsPerLoad + lane / C::kCPR;
    if (fused) {
      const int c = n0 + r;  // interleaved column: gate row c / 2, up row F + c / 2
      wro[g] = c < N ? (uint32_t)((int64_t)((c & 1) ? gg.swiglu_f + (c >> 1) : (c >> 1)) * ld * 2) : kNoRow;
    } else {
      wro[g] = (uint32_t)((int64_t)r * ld * 2);
    }
  }

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{};

  const int nk = (K + BK - 1) / BK;
  auto stage_x = [&](int s) { return smem + s * C::kStageBytes; };
  auto stage_w = [&](int s) { return smem + s * C::kStageBytes + BM * C::kRowBytes; };
  auto load = [&](int kt) {
    load_slice<C, BM>(xr, stage_x(kt % S), xro, K, kt * BK, wave, lane);
    load_slice<C, BN>(wr, stage_w(kt % S), wro, K, kt * BK, wave, lane);
  };

#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (s < nk) load(s);

  // operand lane roles: row fr of a 16-row fragment, 8-k chunk fh of 32
  const int fr = lane & (MI - 1), fh = lane / MI;
  constexpr int KS = BK / 32;  // MFMA k-steps per slice
  // per-lane byte offset of this lane's 16-byte fragment row in k-step ks
  int lane_off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) lane_off[ks] = fr * C::kRowBytes + (((4 * ks + fh) ^ swz<C::kCPR>(fr)) << 4);
  // the x slice sits first in a stage, the W slice after it
  const int x_row0 = wm * WM * C::kRowBytes, w_row0 = BM * C::kRowBytes + wn * WN * C::kRowBytes;

  bf16x8 a[2][TN], b[2][TM];
  auto frags = [&](const OPS_LDS char* st, int ks, int buf) {
#pragma unroll
    for (int i = 0; i < TN; ++i) a[buf][i] = lds_frag<C>(st + w_row0 + i * MI * C::kRowBytes + lane_off[ks]);
#pragma unroll
    for (int j = 0; j < TM; ++j) b[buf][j] = lds_frag<C>(st + x_row0 + j * MI * C::kRowBytes + lane_off[ks]);
  };
  // The MFMAs of the last k-step of slice kt with the loads of slice kt + 2
  // interleaved, one load after each MFMA, so no wave issues its loads in one
  // burst (the issue of a stalled load would hold back the MFMAs behind it).
  // Past the last slice the loads are out of range (they read zeros) and go
  // to the stage no wave reads any more.
  auto mfmas_loading = [&](int buf, int kt) {
    constexpr int MF = TN * TM, L = C::kLoadsPerTile;
    OPS_LDS char* dst = smem + ((kt + 1 < nk ? kt : kt + 1) & 1) * C::kStageBytes;
    const int rl = lane / C::kCPR, pc = lane % C::kCPR;
    const int k0 = (kt + 2) * BK;
    const bool more = kt + 2 < nk;
#pragma unroll
    for (int q = 0; q < (MF > L ? MF : L); ++q) {
      if (q < MF) {
        const int i = q / TM, j = q % TM;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[buf][i], b[buf][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      }
      if (q < L) {
        const bool isx = q < LX;
        const int grp = (isx ? q : q - LX) * C::kWaves + wave;
        const int r = grp * C::kRowsPerLoad + rl;
        const int k = k0 + ((pc ^ swz<C::kCPR>(r)) << 3);
        const uint32_t ro = isx ? xro[q < LX ? q : 0] : wro[q >= LX ? q - LX : 0];
        const uint32_t voff = (more && k < K && ro != kNoRow) ? ro + (uint32_t)k * 2u : kOobOffset;
        buffer_load16_lds<kNoL1>(isx ? xr : wr, dst + (isx ? 0 : BM * C::kRowBytes) + grp * 1024, voff);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
    }
  };
  // The next k-step's fragment reads (issued just before, in the same block)
  // go one after each MFMA: left to itself the scheduler puts them after the
  // MFMAs, and the next k-step then waits for a whole LDS round trip.
  auto mfmas = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[buf][i], b[buf][j], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int q = 0; q < TN * TM; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
      if (q < TN + TM) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
    }
  };

  // vmcnt <= n loads of this wave (n a multiple of kLoadsPerTile, < S slices)
  auto wait_slices = [&](int n) {
    constexpr int L = C::kLoadsPerTile;
    if (n <= 0) wait_vmcnt<0>();
    else if (n == 1) wait_vmcnt<L>();
    else if (n == 2) wait_vmcnt<(S > 2 ? 2 : 1) * L>();
    else wait_vmcnt<(S > 3 ? 3 : 1) * L>();
  };
  if constexpr (C::DEEP) {
    static_assert(S >= 3 && S <= 4, "deep ring of 3 or 4 stages");
    // Slices kt + 1 .. kt + S - 1 are in flight while slice kt is used; the
    // stage of slice kt - 1 is refilled right after the barrier that ends it.
    wait_slices(min(S - 2, nk - 1));
    barrier_keep_loads();
    for (int kt = 0; kt < nk; ++kt) {
      if (kt + S - 1 < nk) load(kt + S - 1);
      const OPS_LDS char* st = smem + (kt % S) * C::kStageBytes;
      frags(st, 0, 0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + 1 < KS) frags(st, ks + 1, (ks + 1) & 1);
        mfmas(ks & 1);
      }
      // slice kt + 1 landed: the loads issued after it stay in flight
      if (kt + 1 < nk) wait_slices(min(S - 2, nk - 2 - kt));
      barrier_keep_loads();
    }
  } else if constexpr (S == 2) {
    // Slice kt + 1 is made visible before the last k-step of slice kt: that
    // step already reads slice kt + 1's first fragments, and the MFMAs issued
    // just before the barrier keep the matrix cores busy while the waves
    // meet.  Slice kt + 2 is then loaded into the stage slice kt used (every
    // wave has read its last fragments of it before the barrier).
    wait_vmcnt<0>();
    __syncthreads();
    if (nk > 1) load(1);
    frags(smem, 0, 0);
    for (int kt = 0; kt < nk; ++kt) {
      const OPS_LDS char* st = smem + (kt & 1) * C::kStageBytes;
      const OPS_LDS char* st_next = smem + ((kt + 1) & 1) * C::kStageBytes;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int nb = (ks + 1) & 1;
        if (ks + 1 < KS) {
          frags(st, ks + 1, nb);
        } else if (kt + 1 < nk) {
          wait_vmcnt<0>();
          __syncthreads();
          frags(st_next, 0, nb);
        }
        if (ks == KS - 1) mfmas_loading(ks & 1, kt);
        else mfmas(ks & 1);
      }
    }
  } else {
    // Look-ahead pipeline: at the top of iteration kt slice kt + 1 is made
    // visible, so the last k-step of slice kt already reads slice kt + 1's
    // first fragments and the matrix cores never wait on the barrier.
    if (S > 2 && nk > S - 2) wait_vmcnt<C::kLoadsPerTile * (S > 2 ? S - 2 : 0)>();
    else wait_vmcnt<0>();
    __syncthreads();
    frags(smem, 0, 0);
    for (int kt = 0; kt < nk; ++kt) {
      if (S > 3 && kt + S - 2 < nk) wait_vmcnt<C::kLoadsPerTile * (S > 3 ? S - 3 : 0)>();
      else wait_vmcnt<0>();
      __syncthreads();
      if (kt + S - 1 < nk) load(kt + S - 1);
      const OPS_LDS char* st = smem + (kt % S) * C::kStageBytes;
      const OPS_LDS char* st_next = smem + ((kt + 1) % S) * C::kStageBytes;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int nb = (ks + 1) & 1;
        if (ks + 1 < KS) frags(st, ks + 1, nb);
        else if (kt + 1 < nk) frags(st_next, 0, nb);
        mfmas(ks & 1);
      }
    }
  }

  wait_vmem();  // no LDS DMA may still be in flight when the workgroup ends

  // Epilogue.  acc[i][j] element e: n = n0 + wn*WN + i*16 + fh*4 + e,
  // m = m0 + wm*WM + j*16 + fr.  Four consecutive n per lane -> one 8-byte store
  // (one 16-byte store of fp32 partials under split-K).
  if (tile_part) {
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int r = wm * WM + j * MI + fr;
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        const int c = wn * WN + i * MI + fh * 4;
        *reinterpret_cast<f32x4*>(tile_part + r * BN + c) = acc[i][j];
      }
    }
    return;
  }
  if (part && tail_cnt == 0) {
    float* pbase = part + (int64_t)split * M * N;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int m = m0 + wm * WM + j * MI + fr;
      if (m - m0 >= m_rows) continue;
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        const int n = n0 + wn * WN + i * MI + fh * 4;
        if (n >= N) continue;
        *reinterpret_cast<f32x4*>(pbase + (int64_t)m * N + n) = acc[i][j];
      }
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int m = m0 + wm * WM + j * MI + fr;
    if (m - m0 >= m_rows) continue;
    if (fused) {
      // two (gate, up) pairs per lane: act[m][n / 2], act[m][n / 2 + 1]
      __bf16* arow = y + (int64_t)m * gg.swiglu_f;
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        const int n = n0 + wn * WN + i * MI + fh * 4;
        if (n >= N) continue;
        const float g0 = acc[i][j][0], u0 = acc[i][j][1], g1 = acc[i][j][2], u1 = acc[i][j][3];
        const float a0 = g0 / (1.f + __expf(-g0)) * u0, a1 = g1 / (1.f + __expf(-g1)) * u1;
        *reinterpret_cast<uint32_t*>(arow + (n >> 1)) = pack_bf2(a0, a1);
      }
      continue;
    }
    __bf16* yrow = y + (int64_t)m * N;
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      {
        const int n = n0 + wn * WN + i * MI + fh * 4;
        if (n >= N) continue;
        float v0 = acc[i][j][0], v1 = acc[i][j][1];
        float v2 = acc[i][j][2], v3 = acc[i][j][3];
        if (bias) {
          const u32x2 bb = *reinterpret_cast<const u32x2*>(bias + n);
          v0 += bf_lo(bb[0]);
          v1 += bf_hi(bb[0]);
          v2 += bf_lo(bb[1]);
          v3 += bf_hi(bb[1]);
        }
        u32x2 out;
        out[0] = pack_bf2(v0, v1);
        out[1] = pack_bf2(v2, v3);
        *reinterpret_cast<u32x2*>(yrow + n) = out;
      }
    }
  }
}

// One MFMA 16x16x32 on an accumulator held in AGPRs.  Issued from inline
// assembly so that the 64 accumulators of a 128x128 wave tile stay in place:
// with the builtin the register allocator rotated them through AGPR copies and
// spilled.  An assembly statement with side effects also fixes the order of
// the memory instructions around it, which places the fragment reads and the
// tile loads between the MFMAs exactly as written.
__device__ __forceinline__ void mfma_agpr(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// An accumulator's four values into VGPRs.  Read through assembly as well:
// were the epilogue's arithmetic to read the AGPRs directly, the compiler
// would give the accumulators VGPR homes and copy them around every MFMA.
__device__ __forceinline__ f32x4 agpr_read(const f32x4& acc) {
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[e]) : "a"(acc[e]));
  return v;
}

// acc <- 0 by a small MFMA on zero operands: the matrix core is idle in the
// epilogue, and the accumulator stays the AGPR tuple it is (zeroed in C++ it
// got VGPR homes and spilled).
__device__ __forceinline__ void agpr_zero(f32x4& acc, const u32x2& zero) {
  asm volatile("v_mfma_f32_4x4x4_16b_f16 %0, %1, %1, 0" : "+a"(acc) : "v"(zero));
}

// Order a scalar or vector value among the other assembly statements: work on
// it between two pins stays between the MFMAs it is written between.
template <class V>
__device__ __forceinline__ void pin_s(V& v) {
  asm volatile("" : "+s"(v));
}
template <class V>
__device__ __forceinline__ void pin_v(V& v) {
  asm volatile("" : "+v"(v));
}

// The 256x256 tile as four waves of 128x128, one wave per SIMD.  With two
// waves per SIMD (gemm_bf16_kernel's eight-wave form) the older wave takes
// the matrix core first and then waits at the slice barrier while the younger
// one finishes alone; here every SIMD runs one wave and the slice's fragment
// reads fall from 192 to 128 KB per workgroup.
//
// What bounds it: one wave issues everything, about one instruction every 4
// cycles, and a 16x16x32 MFMA takes 16, so more than three other instructions
// between two MFMAs leave the matrix core idle.  Hence:
//  * a tile load is two instructions (M0, the load): its per-lane offset is
//    constant, the descriptor's base moves along K once per slice in scalar
//    registers.  (Offsets computed per load in vector registers cost the 8871
//    x 28672 x 4096 gate-up 1587 against 1480 us, the same card.)
//  * a k-step is 64 MFMAs; the 16 fragment reads of the next k-step go one
//    after every second MFMA of the first half, 8 tile loads one after every
//    eighth MFMA (spread over both k-steps of a slice: 1480 -> 1454 us, the
//    14336-long down projection 757 -> 705);
//  * everything else (descriptor, ring and address updates) is pinned between
//    MFMAs, a few instructions at a place; a slice ends in a wait and a branch
//    (1451 -> 1430 us, 16384 x 57344 x 8192 10300 -> 9850).
//
// The LDS ring is five 32 KB half-slices (160 KB) rather than two 64 KB
// slices: the x half and the W half of a slice rotate through the buffers
// separately.  The lead operand's half of slice s + 2 is loaded during the
// first k-step of slice s (into the buffer slice s - 1 freed), the other
// operand's during the second, so 1 to 1.5 slices are in flight per CU.
//
// A workgroup runs a chain of up to kMaxChain tiles: the loads run on into the
// next tile's first slices while the last ones of this tile are used, and the
// stores of a tile drain under the next one's first slice.  A tile of its own
// pays the first loads' latency and the drain each time (about 10 of the 93
// us of a K = 4096 tile).  Chains shorten towards the end of a launch, so that
// it balances over whatever CUs it gets (gemm_schedule.h).
//
// The columns of a W fragment pair are interleaved in runs of four (fragment
// i, row f: column 32 (i / 2) + 8 (f / 4) + 4 (i & 1) + f % 4), so a lane's
// two accumulators hold eight consecutive columns: one 16-byte store.  The W
// rows are swizzled by that row's place in the fragment, as the x rows are.
template <class C, bool XLEAD, bool RAGGED_K, bool GROUPED>
__global__ __launch_bounds__(C::kThreads, 1) void gemm_bf16_w4_kernel(const __bf16* __restrict__ x,
                                                                      const __bf16* __restrict__ W,
                                                                      const __bf16* __restrict__ bias,
                                                                      __bf16* __restrict__ y, int M, int N,
                                                                      int K_total, int group_m, int kchunk,
                                                                      float* __restrict__ part, GroupedGemm gg,
                                                                      int dp_cnt, int tail_cnt, int items,
                                                                      bool chained) {
  static_assert(C::kWaves == 4 && C::WM == 128 && C::WN == 128 && !C::DEEP, "four waves of 128x128");
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, WM = C::WM, WN = C::WN;
  constexpr int MI = 16, TM = WM / MI, TN = WN / MI, KS = BK / 32;
  constexpr int LX = BM / C::kRowsPerLoad / C::kWaves, LW = BN / C::kRowsPerLoad / C::kWaves;
  static_assert(KS == 2, "two k-steps per slice");
  static_assert(BM == BN && LX == 8 && LW == 8, "square tile: x and W halves of 8 loads per wave");
  constexpr int kStores = TM * TN / 2;  // 16-byte stores of a tile per lane
  constexpr uint32_t kOutOfRange = 0xfffffff0u;

  const int tiles_n = (N + BN - 1) / BN;
  const int tiles_m = (M + BM - 1) / BM;
  const int tiles = tiles_m * tiles_n;
  const int ld = K_total;
  const bool fused = GROUPED && gg.swiglu_f > 0;
  if constexpr (GROUPED) items = gg.tiles[gg.E] * tiles_n;  // (the grid is an upper bound)

  // One work item: a tile and its K range.
  struct Item {
    uint64_t xb, wb;      // the tile's first x and W row at the range's first k
    uint32_t xrec, wrec;  // bytes addressable from there: rows past the tile's end read zeros
    int K;                // length of the range
    int m0, n0, m_rows, split;
    float* tile_part;     // split tail: the compact fp32 partial tile
  };
  auto decode = [&](int id) {
    Item it;
    it.split = 0;
    it.tile_part = nullptr;
    int kc = kchunk;
    if constexpr (GROUPED) {
      // items in the order expert, column block, tile-row of the expert
      const int l = (int)xcd_remap((uint32_t)id, (uint32_t)items);
      int lo = 0, hi = gg.E;  // gg.tiles[lo] * tiles_n <= l < gg.tiles[hi] * tiles_n
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (gg.tiles[mid] * tiles_n <= l) lo = mid;
        else hi = mid;
      }
      const int t0 = gg.tiles[lo], tr_e = gg.tiles[lo + 1] - t0;  // tile-rows of expert lo (>= 1)
      const int local = l - t0 * tiles_n;
      const int tn = local / tr_e, tr = local - tn * tr_e;
      it.n0 = tn * BN;
      it.m0 = gg.rows[lo] + tr * BM;
      it.m_rows = min(BM, gg.rows[lo + 1] - it.m0);
      it.K = ld;
      // x: the whole operand (rows are gathered per lane); W: the expert's
      // rows from the tile's first (fused SwiGLU: gate row n0 / 2) on
      it.xb = (uint64_t)(uintptr_t)x;
      it.xrec = (uint32_t)((int64_t)gg.x_rows * ld * 2);
      const int w0 = fused ? it.n0 / 2 : it.n0;
      it.wb = (uint64_t)(uintptr_t)(W + lo * gg.w_stride + (int64_t)w0 * ld);
      it.wrec = (uint32_t)((int64_t)(fused ? N - w0 : min(BN, N - it.n0)) * ld * 2);
      return it;
    }
    uint32_t tid;
    if (tail_cnt == 0) {
      it.split = id / tiles;
      tid = xcd_remap(id - it.split * tiles, (uint32_t)tiles);
    } else if (id < dp_cnt) {
      tid = xcd_remap(id, (uint32_t)dp_cnt);
      kc = K_total;
    } else {
      const int b = id - dp_cnt;
      it.split = b / tail_cnt;
      const int t = (int)xcd_remap(b - it.split * tail_cnt, (uint32_t)tail_cnt);
      tid = dp_cnt + t;
      it.tile_part = part + ((int64_t)it.split * tail_cnt + t) * BM * BN;
    }
    int tm, tn;
    tile_coords(tid, tiles_m, tiles_n, group_m, tm, tn);
    it.m0 = tm * BM;
    it.n0 = tn * BN;
    it.m_rows = min(BM, M - it.m0);
    const int k_begin = it.split * kc;
    it.K = min(K_total - k_begin, kc);
    it.xb = (uint64_t)(uintptr_t)(x + (int64_t)it.m0 * ld + k_begin);
    it.xrec = (uint32_t)(((int64_t)(it.m_rows - 1) * ld + it.K) * 2);
    it.wb = (uint64_t)(uintptr_t)(W + (int64_t)it.n0 * ld + k_begin);
    it.wrec = (uint32_t)(((int64_t)(min(BN, N - it.n0) - 1) * ld + it.K) * 2);
    return it;
  };

  // This workgroup's chain: items id, id + kNumCUs, ... below id_end.
  const Chain ch = chain_of((int)(blockIdx.x / kNumCUs), (items + kNumCUs - 1) / kNumCUs, chained);
  int id = ch.first * kNumCUs + (int)(blockIdx.x % kNumCUs);
  const int id_end = min(items, (ch.first + ch.len) * kNumCUs);
  if (id >= id_end) return;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave % C::WGM, wn = wave / C::WGM;

  // Byte offsets of the rows this lane loads, its 16-byte chunk swizzled: x by
  // row mod 8, W by the row's place in its fragment mod 8.
  const int rl = lane / C::kCPR, pc = lane % C::kCPR;
  const int xc = pc ^ rl, wc = pc ^ ((rl & 3) | ((wave & 1) << 2));
  uint32_t xro[LX], wro[LW];
  auto load_row = [&](int g) { return (g * C::kWaves + wave) * C::kRowsPerLoad + rl; };
#pragma unroll
  for (int g = 0; g < LX; ++g) {
    const int r = load_row(g);
    xro[g] = (uint32_t)(r * ld * 2) + (uint32_t)(xc << 4);
    // (fused SwiGLU: column c is gate row c / 2, or up row F + c / 2 if odd)
    wro[g] = (uint32_t)((int64_t)(fused ? (r & 1) * gg.swiglu_f + (r >> 1) : r) * ld * 2) + (uint32_t)(wc << 4);
  }
  // Grouped: the x rows of an item's tile (-1: none), and their offsets.
  auto gather_rows = [&](const Item& it, int (&src)[LX]) {
#pragma unroll
    for (int g = 0; g < LX; ++g) {
      const int r = load_row(g);
      src[g] = -1;
      if (r < it.m_rows) src[g] = gg.gather ? gg.gather[it.m0 + r] : it.m0 + r;
    }
  };
  auto row_offsets = [&](const int (&src)[LX], uint32_t (&off)[LX]) {
#pragma unroll
    for (int g = 0; g < LX; ++g)
      off[g] = src[g] >= 0 ? (uint32_t)((int64_t)src[g] * ld * 2) + (uint32_t)(xc << 4) : kOutOfRange;
  };
  [[maybe_unused]] uint32_t xnext[LX] = {};  // grouped: offsets of the item the x cursor enters next

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{};

  Item cur = decode(id), nxt;
  if constexpr (GROUPED) {
    int src[LX];
    gather_rows(cur, src);
    row_offsets(src, xro);
  }
  bool has_next = false;
  // The item the load cursors enter next.  (The cursors are at most two
  // slices ahead, so an item followed by another has at least three slices;
  // the launcher sees to it.)
  auto next_item = [&]() {
    id += kNumCUs;
    has_next = id < id_end;
    if (has_next) {
      nxt = decode(id);
    } else {
      // nothing left: every further load is out of range (zeros into buffers
      // no wave reads any more)
      nxt.xb = cur.xb;
      nxt.wb = cur.wb;
      nxt.xrec = nxt.wrec = 0;
      nxt.K = 0x40000000;
    }
  };
  // Load cursors of the lead (l) and the other operand (f): base, records and
  // k left in the item.  A row past the item's end lies past the records
  // whatever the k; k past the range (RAGGED_K) is masked per lane.
  uint64_t lb = XLEAD ? cur.xb : cur.wb, fb = XLEAD ? cur.wb : cur.xb;
  uint32_t lrec = XLEAD ? cur.xrec : cur.wrec, frec = XLEAD ? cur.wrec : cur.xrec;
  int lk = cur.K, fk = cur.K;
  // one slice further, in parts that each fit between two MFMAs
  constexpr int kAdvance = GROUPED ? 3 + LX / 2 : 3;
  [[maybe_unused]] int x_moved = 0;  // grouped: the x cursor entered its next item
  auto advance = [&](auto lead_c, int step) {
    constexpr bool LEAD = decltype(lead_c)::value, ISX = LEAD == XLEAD;
    uint64_t& base = LEAD ? lb : fb;
    uint32_t& rec = LEAD ? lrec : frec;
    int& kl = LEAD ? lk : fk;
    if (step == 0) {
      pin_s(base);
      base += BK * 2;
      pin_s(base);
    } else if (step == 1) {
      pin_s(kl);
      kl -= BK;
      pin_s(kl);
      base = kl > 0 ? base : (ISX ? nxt.xb : nxt.wb);
      pin_s(base);
    } else if (step == 2) {
      pin_s(kl);
      if constexpr (GROUPED && ISX) x_moved = kl > 0 ? 0 : 1;
      rec = kl > 0 ? rec : (ISX ? nxt.xrec : nxt.wrec);
      kl = kl > 0 ? kl : nxt.K;
      pin_s(rec);
      pin_s(kl);
    } else if constexpr (GROUPED && ISX) {
#pragma unroll
      for (int g = 2 * (step - 3); g < 2 * (step - 3) + 2; ++g) {
        pin_v(xro[g]);
        xro[g] = x_moved ? xnext[g] : xro[g];
        pin_v(xro[g]);
      }
    }
  };
  constexpr int HB = BM * C::kRowBytes;
  // load g (0 .. 7) of the cursor's half-slice into LDS buffer dst
  auto load_half = [&](auto lead_c, uint32_t dst, int g) {
    constexpr bool LEAD = decltype(lead_c)::value, ISX = LEAD == XLEAD;
    uint32_t voff = ISX ? xro[g] : wro[g];
    if (RAGGED_K) voff = (ISX ? xc : wc) * 8 < (LEAD ? lk : fk) ? voff : kOutOfRange;
    buffer_load16_lds<kNoL1>(make_rsrc((const void*)(uintptr_t)(LEAD ? lb : fb), LEAD ? lrec : frec),
                             (OPS_LDS char*)(uintptr_t)(dst + (g * C::kWaves + wave) * 1024), voff);
  };
  using LD = std::true_type;   // the lead operand
  using FO = std::false_type;  // the other one

  const int fr = lane & (MI - 1), fh = lane / MI;
  uint32_t x_off[KS], w_off[KS];  // this lane's fragment row and chunk in k-step ks
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int ch = ((4 * ks + fh) ^ (fr & 7)) << 4;
    x_off[ks] = (wm * WM + fr) * C::kRowBytes + ch;
    w_off[ks] = (wn * WN + (fr >> 2) * 8 + (fr & 3)) * C::kRowBytes + ch;
  }
  bf16x8 a[2][TN], b[2][TM];
  uint32_t ax, aw;  // fragment addresses (x, W) of the next reads
  // fragment read r (0 .. TN + TM - 1) of a k-step, in the order the MFMAs (i
  // outer, j inner) first need them: b0, a0, b1 .. b7, a1 .. a7
  auto read_frag = [&](int buf, int r) {
    auto xf = [&](int j) { return lds_frag<C>((const OPS_LDS char*)(uintptr_t)(ax + j * MI * C::kRowBytes)); };
    auto wf = [&](int i) {
      return lds_frag<C>((const OPS_LDS char*)(uintptr_t)(aw + ((i >> 1) * 32 + (i & 1) * 4) * C::kRowBytes));
    };
    if (r == 0) b[buf][0] = xf(0);
    else if (r == 1) a[buf][0] = wf(0);
    else if (r < TM + 1) b[buf][r - 1] = xf(r - 1);
    else a[buf][r - TM] = wf(r - TM);
  };
  // One k-step on fragment buffer BUF: the next one's fragments into the
  // other, the cursor's half-slice into LDS buffer dst, side(q) after MFMA q.
  // Its own fragments have landed (the LDS counter is cleared before it, so
  // the compiler needs no wait inside the run; it could not name one that
  // lets the new reads stay in flight: the counter holds at most 15).
  auto kstep = [&](auto buf_c, auto lead_c, uint32_t dst, auto side) {
    constexpr int buf = decltype(buf_c)::value;
#pragma unroll
    for (int q = 0; q < TN * TM; ++q) {
      mfma_agpr(acc[q / TM][q % TM], a[buf][q / TM], b[buf][q % TM]);
      if (q % 2 == 0 && q / 2 < TN + TM) read_frag(buf ^ 1, q / 2);
      if ((q & 7) == 3) load_half(lead_c, dst, q >> 3);
      side(q);
    }
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;

  // Ring buffers (LDS addresses): c0 and c1 hold the lead and the other half
  // of slice s, c2 and c3 those of slice s + 1, c4 the lead half of slice s + 2.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(OPS_LDS char*)smem_raw;
  uint32_t c0 = lds0, c1 = lds0 + HB, c2 = lds0 + 2 * HB, c3 = lds0 + 3 * HB, c4 = lds0 + 4 * HB;
#pragma unroll
  for (int g = 0; g < LX; ++g) load_half(LD{}, c0, g);
#pragma unroll
  for (int g = 0; g < LX; ++g) load_half(FO{}, c1, g);
  next_item();
  if constexpr (GROUPED) {
    if (has_next) {
      int src[LX];
      gather_rows(nxt, src);
      row_offsets(src, xnext);
    }
  }
#pragma unroll
  for (int p = 0; p < kAdvance; ++p) {
    advance(LD{}, p);
    advance(FO{}, p);
  }
#pragma unroll
  for (int g = 0; g < LX; ++g) load_half(LD{}, c2, g);
#pragma unroll
  for (int g = 0; g < LX; ++g) load_half(FO{}, c3, g);
#pragma unroll
  for (int p = 0; p < kAdvance; ++p) advance(LD{}, p);  // (the other cursor moves in the loop's first k-step)
  wait_vmcnt<2 * LX>();                          // slice 0 has landed
  barrier_keep_loads();
  ax = x_off[0] + (XLEAD ? c0 : c1);
  aw = w_off[0] + (XLEAD ? c1 : c0);
#pragma unroll
  for (int r = 0; r < TN + TM; ++r) read_frag(0, r);
  ax = x_off[1] + (XLEAD ? c0 : c1);
  aw = w_off[1] + (XLEAD ? c1 : c0);
  // the accumulators were zeroed by VALU writes: two wait states before an
  // MFMA reads them (the assembler statement hides them from the compiler)
  asm volatile("s_nop 1" ::);
  int left = (cur.K + BK - 1) / BK;  // slices left of the tile
  int fresh = 0;                     // 1: the previous tile's stores may be in flight
  for (;;) {
    // Past the chain's last slice the same body runs on (loads out of range,
    // look-ahead reads never used): one branch-free MFMA run keeps every
    // accumulator in one place.
    do {
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt unconstrained
      kstep(B0{}, LD{}, c4, [&](int q) {
        if (q == 36) advance(FO{}, 0);
        if (q == 40) advance(FO{}, 1);
        if (q == 48) advance(FO{}, 2);
        if (q > 48 && q < 46 + kAdvance) advance(FO{}, q - 46);
        if (q == 56) {
          ax = x_off[0] + (XLEAD ? c2 : c3);
          pin_v(ax);
        }
        if (q == 57) {
          aw = w_off[0] + (XLEAD ? c3 : c2);
          pin_v(aw);
        }
      });
      // Slice s + 1 has landed in every wave: newer than its loads are the
      // lead half of slice s + 2 and, in a tile's first slice, the stores of
      // the tile before it.  And every wave is done reading slice s, whose
      // buffers take the next loads.
      if (!fresh) wait_vmcnt<LX>();
      else wait_vmcnt<LX + kStores>();
      fresh = 0;
      barrier_keep_loads();
      kstep(B1{}, FO{}, c0, [&](int q) {
        if (q == 36) advance(LD{}, 0);
        if (q == 40) advance(LD{}, 1);
        if (q == 48) advance(LD{}, 2);
        if (q > 48 && q < 46 + kAdvance) advance(LD{}, q - 46);
        if (q == 56) {
          ax = x_off[1] + (XLEAD ? c2 : c3);
          pin_v(ax);
        }
        if (q == 57) {
          aw = w_off[1] + (XLEAD ? c3 : c2);
          pin_v(aw);
        }
        if (q == 60) {
          const uint32_t t0 = c0, t1 = c1;
          c0 = c2;
          c1 = c3;
          c2 = c4;
          c3 = t0;
          c4 = t1;
          pin_s(c0);
          pin_s(c1);
          pin_s(c2);
        }
        if (q == 61) {
          pin_s(c3);
          pin_s(c4);
          --left;
          pin_s(left);
        }
      });
    } while (left > 0);

    // The epilogue's reads of the accumulators follow the last MFMA's writes:
    // a 16-pass XDL write needs up to 19 wait states before another
    // instruction reads its result.
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::);
    // (the lane is made opaque: hoisted out of the item loop, the store
    // addresses would not fit beside the fragments)
    int elane = lane;
    pin_v(elane);
    const int er = elane & (MI - 1), eh = elane / MI;
    // the item after next, its gathered rows requested before the stores
    const bool more = has_next;
    const Item done = cur;
    if (more) {
      cur = nxt;
      next_item();
    }
    [[maybe_unused]] int src[LX];
    if constexpr (GROUPED) {
      if (more && has_next) gather_rows(nxt, src);
    }
    if (!GROUPED && part && (tail_cnt == 0 || done.tile_part)) {
      // fp32 partials: the compact tile of a split tail, or this K range's rows
      float* pb = done.tile_part ? done.tile_part : part + ((int64_t)done.split * M + done.m0) * N + done.n0;
      const int64_t pld = done.tile_part ? BN : N;
      const int rows = done.tile_part ? BM : done.m_rows, cols = done.tile_part ? BN : N - done.n0;
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int r = wm * WM + j * MI + er;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
          const int c = wn * WN + (i >> 1) * 32 + eh * 8 + (i & 1) * 4;
          const f32x4 v = agpr_read(acc[i][j]);
          if (r < rows && c < cols) *reinterpret_cast<f32x4*>(pb + r * pld + c) = v;
        }
      }
    } else {
      // exactly kStores stores per wave, whatever the tile's edges (out of
      // range ones are dropped): the wait above counts them
      fresh = 1;
      const int half = fused ? 1 : 0;  // fused SwiGLU: two columns make one activation
      const int ny = N >> half;
      const __amdgpu_buffer_rsrc_t yr =
          make_rsrc(y + (int64_t)done.m0 * ny + (done.n0 >> half),
                    (uint32_t)(((int64_t)(done.m_rows - 1) * ny + ny - (done.n0 >> half)) * 2));
      const int c0e = wn * WN + eh * 8;
      u32x4 bb[TN / 2] = {};
      if (!GROUPED && bias) {
#pragma unroll
        for (int p = 0; p < TN / 2; ++p)
          if (done.n0 + c0e + p * 32 < N) bb[p] = *reinterpret_cast<const u32x4*>(bias + done.n0 + c0e + p * 32);
      }
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int r = wm * WM + j * MI + er;
        const uint32_t row = (uint32_t)(r * ny + (c0e >> half)) * 2u;
#pragma unroll
        for (int p = 0; p < TN / 2; ++p) {
          f32x4 lo = agpr_read(acc[2 * p][j]), hi = agpr_read(acc[2 * p + 1][j]);
          if (!GROUPED && bias) {
            lo += f32x4{bf_lo(bb[p][0]), bf_hi(bb[p][0]), bf_lo(bb[p][1]), bf_hi(bb[p][1])};
            hi += f32x4{bf_lo(bb[p][2]), bf_hi(bb[p][2]), bf_lo(bb[p][3]), bf_hi(bb[p][3])};
          }
          const uint32_t off = r < done.m_rows && done.n0 + c0e + p * 32 < N ? row + (p * 64 >> half) : kOutOfRange;
          if (fused) {
            auto act = [](float g, float u) { return g / (1.f + __expf(-g)) * u; };
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{pack_bf2(act(lo[0], lo[1]), act(lo[2], lo[3])),
                                                        pack_bf2(act(hi[0], hi[1]), act(hi[2], hi[3]))},
                                                  yr, off, 0, 0);
          } else {
            __builtin_amdgcn_raw_buffer_store_b128(
                u32x4{pack_bf2(lo[0], lo[1]), pack_bf2(lo[2], lo[3]), pack_bf2(hi[0], hi[1]), pack_bf2(hi[2], hi[3])},
                yr, off, 0, 0);
          }
        }
      }
    }
    if (!more) break;
    if constexpr (GROUPED) {
      if (has_next) row_offsets(src, xnext);
    }
    u32x2 zero = {0u, 0u};
    pin_v(zero);
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j) agpr_zero(acc[i][j], zero);
    left = (cur.K + BK - 1) / BK;
    asm volatile("s_nop 7" ::);  // (the last zeroes are written before an MFMA reads them)
  }
  wait_vmem();  // no LDS DMA may still be in flight when the workgroup ends
}

// A 128x256 tile as four waves of 128x64 (each all the tile's rows and 64 of its
// columns), for the sizes where 256x256 tiles are too few: decode batches past
// 128 rows and chunks of a few hundred.  Loads, fragments and bookkeeping are
// the four-wave 256x256 kernel's; the LDS (160 KB) holds rings of four x slices
// and three W slices, so up to 112 KB are in flight per CU.  What bounds it is
// the LDS (a slice moves 96 KB of fragments and 48 KB of loads per 1024 cycles
// of MFMAs) and, below 256 rows, the weight stream.  Unsplit launches start
// each column tile at another slice of K and wrap around: in step, all tiles
// would read the same few HBM channels (128 x 28672 x 4096: 68.7 -> 55.1 us); K
// ranges already differ.
// us, the 256x256, 128x256 and 256x128 tiles used before -> this one: 256 x 6144 x
// 4096 32.0 -> 28.1, 256 x 28672 x 4096 87 -> 63, 256 x 4096 x 14336 50.5 -> 45.3, 256
// x 10240 x 8192 70.5 -> 55.4, 512 x 4096 x 4096 41.3 -> 31.2, 1023 x 4096 x 4096 49.7 ->
// 43.8.
template <bool RAGGED_K>
__global__ __launch_bounds__(256, 1) void gemm_bf16_h4_kernel(const __bf16* __restrict__ x,
                                                              const __bf16* __restrict__ W,
                                                              const __bf16* __restrict__ bias,
                                                              __bf16* __restrict__ y, int M, int N, int K_total,
                                                              int group_m, int kchunk,
                                                              float* __restrict__ part) {
  using C = CfgW4;  // (row and chunk geometry of an LDS row)
  constexpr int BM = 128, BN = 256, BK = 64, WM = 128, WN = 64;
  constexpr int MI = 16, TM = WM / MI, TN = WN / MI, KS = 2;  // 8 x 4 MFMA tiles per wave
  constexpr int kWaves = 4, LX = 4, LW = 8;                    // loads per wave of an x / W slice
  constexpr int XS = 4;                                        // ring of x slices (of W's: three)
  constexpr int XB = BM * 128, WB = BN * 128;
  constexpr uint32_t kOutOfRange = 0xfffffff0u;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];

  const int tiles_n = (N + BN - 1) / BN, tiles_m = (M + BM - 1) / BM, tiles = tiles_m * tiles_n;
  const int ld = K_total;
  const int split = blockIdx.x / tiles;
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x - split * tiles, (uint32_t)tiles), tiles_m, tiles_n, group_m, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN, m_rows = min(BM, M - m0);
  const int k_begin = split * kchunk, K = min(K_total - k_begin, kchunk);
  const int nk = (K + BK - 1) / BK;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wn = wave;

  const int rl = lane / 8, pc = lane % 8;
  const int xc = pc ^ rl, wc = pc ^ ((rl & 3) | ((wave & 1) << 2));
  uint32_t xro[LX], wro[LW];
#pragma unroll
  for (int g = 0; g < LX; ++g) xro[g] = (uint32_t)(((g * kWaves + wave) * 8 + rl) * ld * 2) + (uint32_t)(xc << 4);
#pragma unroll
  for (int g = 0; g < LW; ++g) wro[g] = (uint32_t)(((g * kWaves + wave) * 8 + rl) * ld * 2) + (uint32_t)(wc << 4);

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{};

  // the slice this tile starts at
  const int rot = kchunk < K_total ? 0 : tiles_n <= 65536 ? (int)((uint32_t)(tn * nk) / (uint32_t)tiles_n) : tn % nk;
  // Load cursors of x and W: base, records (none once every slice is loaded:
  // the rest read zeros into buffers no wave reads any more), slices left,
  // slices until the wrap to the range's first, k left in the range.
  struct Cursor {
    uint64_t first, base;
    uint32_t rec;
    int left, wrap, k;
  };
  auto cursor = [&](const __bf16* p, int rows) {
    const uint64_t first = (uint64_t)(uintptr_t)(p + k_begin);
    return Cursor{first, first + (uint32_t)rot * (BK * 2), (uint32_t)(((int64_t)(rows - 1) * ld + K) * 2), nk, nk - rot,
                  K - rot * BK};
  };
  Cursor cx = cursor(x + (int64_t)m0 * ld, m_rows), cw = cursor(W + (int64_t)n0 * ld, min(BN, N - n0));
  // one slice further, in two parts that each fit between two MFMAs
  auto advance = [&](Cursor& c, int step) {
    if (step == 0) {
      pin_s(c.base);
      c.base += BK * 2;
      --c.wrap;
      --c.left;
      if (RAGGED_K) c.k -= BK;
      pin_s(c.base);
      pin_s(c.wrap);
      pin_s(c.left);
    } else {
      pin_s(c.wrap);
      c.base = c.wrap > 0 ? c.base : c.first;
      if (RAGGED_K) c.k = c.wrap > 0 ? c.k : K;
      c.wrap = c.wrap > 0 ? c.wrap : 0x40000000;
      c.rec = c.left > 0 ? c.rec : 0;
      pin_s(c.base);
      pin_s(c.wrap);
      pin_s(c.rec);
    }
  };
  auto load = [&](const Cursor& c, uint32_t voff, int chunk, uint32_t dst, int g) {
    if (RAGGED_K) voff = chunk * 8 < c.k ? voff : kOutOfRange;
    buffer_load16_lds<kNoL1>(make_rsrc((const void*)(uintptr_t)c.base, c.rec),
                             (OPS_LDS char*)(uintptr_t)(dst + (g * kWaves + wave) * 1024), voff);
  };
  auto load_x = [&](uint32_t dst, int g) { load(cx, xro[g], xc, dst, g); };
  auto load_w = [&](uint32_t dst, int g) { load(cw, wro[g], wc, dst, g); };

  const int fr = lane & 15, fh = lane >> 4;
  uint32_t x_off[KS], w_off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int ch = ((4 * ks + fh) ^ (fr & 7)) << 4;
    x_off[ks] = fr * 128 + ch;
    w_off[ks] = (wn * WN + (fr >> 2) * 8 + (fr & 3)) * 128 + ch;
  }
  bf16x8 a[2][TN], b[2][TM];
  uint32_t ax, aw;
  auto read_frag = [&](int buf, int r) {
    auto xf = [&](int j) { return lds_frag<C>((const OPS_LDS char*)(uintptr_t)(ax + j * MI * 128)); };
    auto wf = [&](int i) { return lds_frag<C>((const OPS_LDS char*)(uintptr_t)(aw + ((i >> 1) * 32 + (i & 1) * 4) * 128)); };
    if (r == 0) b[buf][0] = xf(0);
    else if (r == 1) a[buf][0] = wf(0);
    else if (r < TM + 1) b[buf][r - 1] = xf(r - 1);
    else a[buf][r - TM] = wf(r - TM);
  };
  auto kstep = [&](auto buf_c, auto side) {
    constexpr int buf = decltype(buf_c)::value;
#pragma unroll
    for (int q = 0; q < TN * TM; ++q) {
      mfma_agpr(acc[q / TM][q % TM], a[buf][q / TM], b[buf][q % TM]);
      if (q % 2 == 0 && q / 2 < TN + TM) read_frag(buf ^ 1, q / 2);
      side(q);
    }
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(OPS_LDS char*)smem_raw;
  // x buffers of slices s .. s + 3, W buffers of slices s .. s + 2
  uint32_t x0 = lds0, x1 = lds0 + XB, x2 = lds0 + 2 * XB, x3 = lds0 + 3 * XB;
  uint32_t w0 = lds0 + XS * XB, w1 = w0 + WB, w2 = w0 + 2 * WB;
  // X(0), W(0), X(1), W(1), X(2), W(2), the order the loop goes on in
#pragma unroll
  for (int s = 0; s < 3; ++s) {
#pragma unroll
    for (int g = 0; g < LX; ++g) load_x(s == 0 ? x0 : s == 1 ? x1 : x2, g);
    advance(cx, 0);
    advance(cx, 1);
#pragma unroll
    for (int g = 0; g < LW; ++g) load_w(s == 0 ? w0 : s == 1 ? w1 : w2, g);
    advance(cw, 0);
    advance(cw, 1);
  }
  wait_vmcnt<2 * (LX + LW)>();
  barrier_keep_loads();
  ax = x_off[0] + x0;
  aw = w_off[0] + w0;
#pragma unroll
  for (int r = 0; r < TN + TM; ++r) read_frag(0, r);
  ax = x_off[1] + x0;
  aw = w_off[1] + w0;
  asm volatile("s_nop 1" ::);
  int left = nk;
  do {
    __builtin_amdgcn_s_waitcnt(0xC07F);
    // k-step 0 of slice s: loads X(s + 3) into x3
    kstep(B0{}, [&](int q) {
      if ((q & 7) == 3) load_x(x3, q >> 3);
      if (q == 28) advance(cx, 0);
      if (q == 29) advance(cx, 1);
      if (q == 30) {
        ax = x_off[0] + x1;
        pin_v(ax);
      }
      if (q == 31) {
        aw = w_off[0] + w1;
        pin_v(aw);
      }
    });
    // slice s + 1 has landed: newer are X(s + 2), W(s + 2), X(s + 3)
    wait_vmcnt<2 * LX + LW>();
    barrier_keep_loads();
    // k-step 1: W(s + 3) into w0 (slice s is read)
    kstep(B1{}, [&](int q) {
      if ((q & 3) == 1) load_w(w0, q >> 2);
      if (q == 26) {
        const uint32_t t = x0;
        x0 = x1;
        x1 = x2;
        x2 = x3;
        x3 = t;
        pin_s(x0);
        pin_s(x1);
        pin_s(x2);
        pin_s(x3);
      }
      if (q == 28) {
        ax = x_off[1] + x0;
        pin_v(ax);
      }
      if (q == 29) {
        aw = w_off[1] + w1;
        pin_v(aw);
        --left;
        pin_s(left);
      }
      if (q == 30) advance(cw, 0);
      if (q == 31) {
        advance(cw, 1);
        const uint32_t t = w0;
        w0 = w1;
        w1 = w2;
        w2 = t;
        pin_s(w0);
        pin_s(w1);
        pin_s(w2);
      }
    });
  } while (left > 0);
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::);
  const int c0 = wn * WN + fh * 8;
  if (part) {
    float* pb = part + ((int64_t)split * M + m0) * N + n0;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int r = j * MI + fr;
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        const int c = c0 + (i >> 1) * 32 + (i & 1) * 4;
        const f32x4 v = agpr_read(acc[i][j]);
        if (r < m_rows && c < N - n0) *reinterpret_cast<f32x4*>(pb + (int64_t)r * N + c) = v;
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int r = j * MI + fr;
#pragma unroll
      for (int p = 0; p < TN / 2; ++p) {
        f32x4 lo = agpr_read(acc[2 * p][j]), hi = agpr_read(acc[2 * p + 1][j]);
        const int n = n0 + c0 + p * 32;
        if (r >= m_rows || n >= N) continue;
        if (bias) {
          const u32x4 bb = *reinterpret_cast<const u32x4*>(bias + n);
          lo += f32x4{bf_lo(bb[0]), bf_hi(bb[0]), bf_lo(bb[1]), bf_hi(bb[1])};
          hi += f32x4{bf_lo(bb[2]), bf_hi(bb[2]), bf_lo(bb[3]), bf_hi(bb[3])};
        }
        *reinterpret_cast<u32x4*>(y + (int64_t)(m0 + r) * N + n) =
            u32x4{pack_bf2(lo[0], lo[1]), pack_bf2(lo[2], lo[3]), pack_bf2(hi[0], hi[1]), pack_bf2(hi[2], hi[3])};
      }
    }
  }
  wait_vmem();
}

// y[m][n] = bf16(sum over splits s of part[s][m][n] (in split order) + bias[n]),
// four consecutive elements per thread (N is a multiple of 8).  BATCH ranges'
// partials are requested together: eight for outputs of at most a workgroup per
// CU, which wait on latency (48 x 4096 over 8 ranges: 0.7 us less), one at a
// time for larger ones, which have other waves to run (256 x 4096: 0.6 less).
template <int BATCH>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int splits,
                                                            const __bf16* __restrict__ bias,
                                                            __bf16* __restrict__ y, int64_t MN, int N) {
  const int64_t n4 = MN / 4;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
    f32x4 a = reinterpret_cast<const f32x4*>(part)[i];
    for (int s0 = 1; s0 < splits; s0 += BATCH) {
      f32x4 v[BATCH];
#pragma unroll
      for (int j = 0; j < BATCH; ++j)
        if (s0 + j < splits) v[j] = reinterpret_cast<const f32x4*>(part + (int64_t)(s0 + j) * MN)[i];
#pragma unroll
      for (int j = 0; j < BATCH; ++j)
        if (s0 + j < splits) a += v[j];
    }
    if (bias) {
      const int n = (int)((i * 4) % N);
      const u32x2 bb = *reinterpret_cast<const u32x2*>(bias + n);
      a[0] += bf_lo(bb[0]);
      a[1] += bf_hi(bb[0]);
      a[2] += bf_lo(bb[1]);
      a[3] += bf_hi(bb[1]);
    }
    reinterpret_cast<u32x2*>(y)[i] = u32x2{pack_bf2(a[0], a[1]), pack_bf2(a[2], a[3])};
  }
}

// y of the split tail: tile dp_cnt + t is the sum over splits (in order) of
// its compact partials, plus bias.  Grid (tail_cnt, BM / 16): 16 rows of one
// tile per workgroup, four consecutive columns per thread (N % 8 == 0).
template <int BM, int BN>
__global__ __launch_bounds__(256) void splitk_tile_reduce_kernel(const float* __restrict__ part, int splits,
                                                                 int dp_cnt, int tail_cnt, int M, int N,
                                                                 int tiles_m, int tiles_n, int group_m,
                                                                 const __bf16* __restrict__ bias,
                                                                 __bf16* __restrict__ y) {
  const int t = blockIdx.x;
  int tm, tn;
  tile_coords(dp_cnt + t, tiles_m, tiles_n, group_m, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  constexpr int C4 = BN / 4;
  for (int idx = threadIdx.x; idx < 16 * C4; idx += 256) {
    const int r = blockIdx.y * 16 + idx / C4, c = (idx % C4) * 4;
    const int m = m0 + r, n = n0 + c;
    if (m >= M || n >= N) continue;
    const float* p = part + (int64_t)t * BM * BN + r * BN + c;
    f32x4 a = *reinterpret_cast<const f32x4*>(p);
    for (int sp = 1; sp < splits; ++sp) a += *reinterpret_cast<const f32x4*>(p + (int64_t)sp * tail_cnt * BM * BN);
    if (bias) {
      const u32x2 bb = *reinterpret_cast<const u32x2*>(bias + n);
      a[0] += bf_lo(bb[0]);
      a[1] += bf_hi(bb[0]);
      a[2] += bf_lo(bb[1]);
      a[3] += bf_hi(bb[1]);
    }
    *reinterpret_cast<u32x2*>(y + (int64_t)m * N + n) = u32x2{pack_bf2(a[0], a[1]), pack_bf2(a[2], a[3])};
  }
}

// Tile-rows per group of the tile order (tile_coords): as many as keep the
// group's x rows (BM x K bf16 each) within kGroupBytes, so they stay in the
// last-level cache while the group sweeps the tile-columns; at least
// kMinGroupRows, at most all.  The floor matters for long K: an XCD runs 32
// consecutive tiles at once, which with one tile-row per group are 1 x 32
// tiles (all of W's column blocks, re-read by every XCD) and with four are
// 4 x 8.  Measured on the 16384 x 8192 x 28672 down projection: 6590 us with
// one row per group, 5550 with two, 5480 with four, 5640 with eight.
constexpr int64_t kMinGroupRows = 4;
template <class C>
static int tile_group_rows(int64_t tiles_m, int64_t tiles_n, int64_t K) {
  (void)tiles_n;
  const int64_t row_block_bytes = (int64_t)C::BM * K * 2;
  return (int)std::max<int64_t>(1, std::min<int64_t>(tiles_m, std::max(kMinGroupRows, kGroupBytes / row_block_bytes)));
}

// K range of one split: a whole number of BK slices; the number of ranges
// that actually results (at most `splits`).
static int64_t split_chunk(int64_t K, int splits, int BK) { return ((K + splits - 1) / splits + BK - 1) / BK * BK; }
static int split_ranges(int64_t K, int splits, int BK) {
  const int64_t c = split_chunk(K, splits, BK);
  return (int)((K + c - 1) / c);
}

// splits > 1: every tile runs as that many K ranges (fp32 partials [splits, M,
// N] in `part`, then an ordered reduce).  tail_splits > 1: only the tiles of
// the last, partly filled round run split (compact fp32 partial tiles in
// `part`), the other tiles as usual in the same launch.  `part` is the
// caller's workspace, sized by plan_linear.
template <class C>
static hipError_t launch_gemm_bf16(const void* x, const void* W, const void* bias, void* y, int64_t M,
                                   int64_t N, int64_t K, hipStream_t s, int splits, int tail_splits, float* part) {
  // More than 64 KB of dynamic LDS per workgroup needs the limit raised once
  // per process (a host-side function attribute, no allocation).
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_kernel<C, false>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, C::kLdsBytes);
  if (attr != hipSuccess) return attr;
  const int64_t tiles_m = (M + C::BM - 1) / C::BM;
  const int64_t tiles_n = (N + C::BN - 1) / C::BN;
  const int64_t tiles = tiles_m * tiles_n;
  const int group_m = tile_group_rows<C>(tiles_m, tiles_n, K);
  const auto kern = &gemm_bf16_kernel<C, false>;
  if (tail_splits > 1) {
    const int64_t tail = tiles % kNumCUs, dp = tiles - tail;
    const int64_t kchunk = split_chunk(K, tail_splits, C::BK);
    const int nsplit = split_ranges(K, tail_splits, C::BK);
    hipLaunchKernelGGL(kern, dim3((unsigned)(dp + tail * nsplit)), dim3(C::kThreads), C::kLdsBytes,
                       s, static_cast<const __bf16*>(x), static_cast<const __bf16*>(W),
                       static_cast<const __bf16*>(bias), static_cast<__bf16*>(y), (int)M, (int)N, (int)K, group_m,
                       (int)kchunk, part, GroupedGemm{}, (int)dp, (int)tail);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((splitk_tile_reduce_kernel<C::BM, C::BN>), dim3((unsigned)tail, C::BM / 16), dim3(256), 0, s,
                       static_cast<const float*>(part), nsplit, (int)dp, (int)tail, (int)M, (int)N, (int)tiles_m,
                       (int)tiles_n, group_m, static_cast<const __bf16*>(bias), static_cast<__bf16*>(y));
    return hipGetLastError();
  }
  const bool split = splits > 1;
  const int64_t kchunk = split ? split_chunk(K, splits, C::BK) : K;
  const int nsplit = split ? split_ranges(K, splits, C::BK) : 1;
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * nsplit)), dim3(C::kThreads), C::kLdsBytes, s,
                     static_cast<const __bf16*>(x), static_cast<const __bf16*>(W),
                     static_cast<const __bf16*>(bias), static_cast<__bf16*>(y), (int)M, (int)N, (int)K,
                     group_m, (int)kchunk, split ? part : nullptr, GroupedGemm{}, 0, 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !split) return e;
  return launch_splitk_reduce(part, nsplit, bias, y, M, N, s);
}

// The same launches on the four-wave kernel: items (tiles, then the K ranges
// of a split tail, or the ranges of every tile), chained where `chained`.
template <bool XLEAD, bool RAGGED_K, bool GROUPED>
static hipError_t launch_gemm_w4_kernel(const void* x, const void* W, const void* bias, void* y, int64_t M, int64_t N,
                                        int64_t K, int group_m, int64_t kchunk, float* part, int64_t dp, int64_t tail,
                                        int64_t items, bool chained, const GroupedGemm& gg, hipStream_t s) {
  using C = CfgW4;
  constexpr int kLds = 5 * C::BM * C::kRowBytes;  // five half-slices
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_w4_kernel<C, XLEAD, RAGGED_K, GROUPED>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return attr;
  const int64_t grid = chain_grid(items, chained, !GROUPED);
  hipLaunchKernelGGL((gemm_bf16_w4_kernel<C, XLEAD, RAGGED_K, GROUPED>), dim3((unsigned)grid), dim3(C::kThreads), kLds, s,
                     static_cast<const __bf16*>(x), static_cast<const __bf16*>(W), static_cast<const __bf16*>(bias),
                     static_cast<__bf16*>(y), (int)M, (int)N, (int)K, group_m, (int)kchunk, part, gg, (int)dp,
                     (int)tail, (int)items, chained);
  return hipGetLastError();
}

static hipError_t launch_gemm_w4(const void* x, const void* W, const void* bias, void* y, int64_t M, int64_t N,
                                 int64_t K, hipStream_t s, int splits, int tail_splits, float* part) {
  using C = CfgW4;
  const int64_t tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN, tiles = tiles_m * tiles_n;
  const int group_m = tile_group_rows<C>(tiles_m, tiles_n, K);
  const int64_t tail = tail_splits > 1 ? tiles % kNumCUs : 0, dp = tiles - tail;
  const int sp = tail ? tail_splits : std::max(1, splits);
  const int64_t kchunk = sp > 1 ? split_chunk(K, sp, C::BK) : K;
  const int nsplit = sp > 1 ? split_ranges(K, sp, C::BK) : 1;
  const int64_t items = tail ? dp + tail * nsplit : tiles * nsplit;
  // the kernel's load cursors run two slices ahead, into the next item only:
  // items of fewer than three slices are not chained
  const bool chained = K - (nsplit - 1) * kchunk > 2 * C::BK;
  // The ring gives half a slice more of lead to one operand: the one with
  // fewer distinct blocks among the 32 tiles an XCD runs at once (x when a
  // group spans at most 4 tile-rows, i.e. K >= 8192; W for the 8-row groups of
  // K = 4096).  On one card, flushed, measured on the ring's first form: the 8B
  // gate-up 1579 -> 1526 us with W leading, down 769 -> 752 us and the 70B
  // gate-up and down 3-4 % faster with x leading.
  const bool xlead = group_m <= 4, ragged = K % C::BK != 0;
  const auto go = [&](auto xl, auto rk) {
    return launch_gemm_w4_kernel<decltype(xl)::value, decltype(rk)::value, false>(
        x, W, bias, y, M, N, K, group_m, kchunk, sp > 1 ? part : nullptr, tail ? dp : 0, tail, items, chained,
        GroupedGemm{}, s);
  };
  using T = std::true_type;
  using F = std::false_type;
  const hipError_t e = xlead ? (ragged ? go(T{}, T{}) : go(T{}, F{})) : (ragged ? go(F{}, T{}) : go(F{}, F{}));
  if (e != hipSuccess || sp == 1) return e;
  if (!tail) return launch_splitk_reduce(part, nsplit, bias, y, M, N, s);
  hipLaunchKernelGGL((splitk_tile_reduce_kernel<C::BM, C::BN>), dim3((unsigned)tail, C::BM / 16), dim3(256), 0, s,
                     static_cast<const float*>(part), nsplit, (int)dp, (int)tail, (int)M, (int)N, (int)tiles_m,
                     (int)tiles_n, group_m, static_cast<const __bf16*>(bias), static_cast<__bf16*>(y));
  return hipGetLastError();
}

// The 128x256 tile: tiles, or splits K ranges of each.
constexpr int kH4Rows = 128, kH4Cols = 256;
static hipError_t launch_gemm_h4(const void* x, const void* W, const void* bias, void* y, int64_t M, int64_t N,
                                 int64_t K, hipStream_t s, int splits, float* part) {
  constexpr int kLds = (4 * kH4Rows + 3 * kH4Cols) * 128;  // rings of four x and three W slices
  static const hipError_t attr = [] {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_h4_kernel<false>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    return e != hipSuccess ? e
                           : hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_h4_kernel<true>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  }();
  if (attr != hipSuccess) return attr;
  const int64_t tiles_m = (M + kH4Rows - 1) / kH4Rows, tiles_n = (N + kH4Cols - 1) / kH4Cols;
  const int64_t kchunk = splits > 1 ? split_chunk(K, splits, 64) : K;
  const int nsplit = splits > 1 ? split_ranges(K, splits, 64) : 1;
  const int group_m = (int)std::min<int64_t>(tiles_m, std::max<int64_t>(2 * kMinGroupRows, kGroupBytes / (kH4Rows * K * 2)));
  const auto kern = K % 64 ? &gemm_bf16_h4_kernel<true> : &gemm_bf16_h4_kernel<false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n * nsplit)), dim3(256), kLds, s,
                     static_cast<const __bf16*>(x), static_cast<const __bf16*>(W), static_cast<const __bf16*>(bias),
                     static_cast<__bf16*>(y), (int)M, (int)N, (int)K, group_m, (int)kchunk,
                     nsplit > 1 ? part : nullptr);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || nsplit <= 1) return e;
  return launch_splitk_reduce(part, nsplit, bias, y, M, N, s);
}

hipError_t launch_splitk_reduce(const float* part, int splits, const void* bias, void* y, int64_t M, int64_t N,
                                hipStream_t s) {
  const int64_t MN = M * N;
  const unsigned blocks = (unsigned)std::min<int64_t>(4096, (MN / 4 + 255) / 256);
  const auto kern = blocks <= (unsigned)kNumCUs ? &splitk_reduce_kernel<8> : &splitk_reduce_kernel<1>;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, s, part, splits, static_cast<const __bf16*>(bias),
                     static_cast<__bf16*>(y), MN, (int)N);
  return hipGetLastError();
}

// Split-K for small M: when at most half as many bm x bn tiles as CUs exist, K
// is cut into floor(kNumCUs / tiles) ranges (each at least 512 wide), so about
// kNumCUs workgroups run.  (A split that only lifts 129-255 tiles a little past
// the CU count measured slower than no split.)  0: no split.
static int splitk_count(int bm, int bn, int64_t M, int64_t N, int64_t K) {
  if (M > kSplitKMaxM || K < 1024) return 0;
  const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  const int64_t s = std::min<int64_t>(kNumCUs / tiles, K / 512);
  return s >= 2 ? (int)s : 0;
}

template <class C>
static hipError_t launch_grouped(const void* x, int64_t x_rows, const void* W, int64_t w_stride, void* y,
                                 int64_t max_rows, int64_t N, int64_t K, int32_t E, const int32_t* gather,
                                 const int32_t* rows, const int32_t* tiles, int32_t swiglu_f, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(gemm_bf16_kernel<C, true>), hipFuncAttributeMaxDynamicSharedMemorySize,
      C::kLdsBytes);
  if (attr != hipSuccess) return attr;
  // at most ceil(rows / BM) + E tile-rows; workgroups past the list's end return
  const int64_t tile_rows = (max_rows + C::BM - 1) / C::BM + E;
  const int64_t tiles_n = (N + C::BN - 1) / C::BN;
  GroupedGemm gg{gather, rows, tiles, E, (int)x_rows, w_stride, swiglu_f};
  hipLaunchKernelGGL((gemm_bf16_kernel<C, true>), dim3((unsigned)(tile_rows * tiles_n)), dim3(C::kThreads),
                     C::kLdsBytes, s, static_cast<const __bf16*>(x), static_cast<const __bf16*>(W), nullptr,
                     static_cast<__bf16*>(y), (int)max_rows, (int)N, (int)K, 1, (int)K, nullptr, gg, 0, 0);
  return hipGetLastError();
}

int32_t grouped_gemm_tile_rows(int64_t rows, int32_t E) {
  // about 64 rows or fewer per expert (decode batches): 64-row tiles, so the
  // matrix cores do not spend most of a 256-row tile on padding; beyond, the
  // four-wave kernel's tiles, which read each expert's weights once where
  // 64-row ones read them twice (us, 64 / 256 rows, 64 experts of 2560, top-8: 56
  // rows an expert 689 / 724, 75 rows 840 / 743, 96 rows 884 / 763; 8 experts of
  // 14336, top-2: 75 rows 699 / 708, 150 rows 1049 / 714)
  return rows <= (int64_t)64 * E ? CfgRow64::BM : CfgBig8::BM;
}

hipError_t launch_gemm_grouped(const void* x, int64_t x_rows, const void* W, int64_t w_stride, void* y,
                               int64_t max_rows, int64_t N, int64_t K, int32_t E, int32_t tile_rows,
                               const int32_t* gather, const int32_t* rows, const int32_t* tiles, int32_t swiglu_f,
                               hipStream_t s) {
  // Decode batches: one workgroup per CU with a deep ring, or two with a shallow one.
  if (tile_rows == CfgRow64::BM) {
    const bool deep = grouped_deep_ring(max_rows, N, E, stream_cus(s));
    return deep ? launch_grouped<CfgSk64>(x, x_rows, W, w_stride, y, max_rows, N, K, E, gather, rows, tiles, swiglu_f, s)
                : launch_grouped<CfgRow64>(x, x_rows, W, w_stride, y, max_rows, N, K, E, gather, rows, tiles, swiglu_f,
                                           s);
  }
  // Large batches: the four-wave kernel (the lead operand as in launch_gemm_w4).
  // 8871 tokens, top-2 of 8 experts, 4096 wide: gate-up with its SwiGLU (14336
  // wide) 3700 -> 3150 us, down 1990 -> 1600, against the eight-wave form.
  // The eight-wave form takes what its chains and 32-bit offsets do not: K of
  // less than three slices, N of 2^22 and more.
  if (K > 2 * CfgW4::BK && N < kW4MaxN) {
    const int64_t tile_rows_max = (max_rows + CfgW4::BM - 1) / CfgW4::BM + E;
    const int64_t items = tile_rows_max * ((N + CfgW4::BN - 1) / CfgW4::BN);
    const GroupedGemm gg{gather, rows, tiles, E, (int)x_rows, w_stride, swiglu_f};
    const auto go = [&](auto xl, auto rk) {
      return launch_gemm_w4_kernel<decltype(xl)::value, decltype(rk)::value, true>(
          x, W, nullptr, y, max_rows, N, K, 1, K, nullptr, 0, 0, items, true, gg, s);
    };
    using T = std::true_type;
    using F = std::false_type;
    const bool ragged = K % CfgW4::BK != 0;
    return K >= 8192 ? (ragged ? go(T{}, T{}) : go(T{}, F{})) : (ragged ? go(F{}, T{}) : go(F{}, F{}));
  }
  return launch_grouped<CfgBig8>(x, x_rows, W, w_stride, y, max_rows, N, K, E, gather, rows, tiles, swiglu_f, s);
}

// The tiled configurations a plan can name.
enum TileCfg { kCfgBig8 = 0, kCfgT192 = 1, kCfgMid = 2, kCfgSk64 = 3, kCfgSk128 = 4, kCfgW4 = 5, kCfgH4 = 6 };

// workspace of a K split (64-wide slices), and of a split tail of bm x bn tiles
static size_t split_bytes(int64_t M, int64_t N, int64_t K, int splits) {
  return (size_t)split_ranges(K, splits, 64) * M * N * sizeof(float);
}
static size_t tail_bytes(int bm, int bn, int64_t M, int64_t N, int64_t K, int tail_splits) {
  const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  return (size_t)split_ranges(K, tail_splits, 64) * (tiles % kNumCUs) * bm * bn * sizeof(float);
}

// Does the small-M kernel's extra reading of x (from L2, 15 TB/s) cost less than
// what the streaming kernel adds: a second launch where it splits K, and a
// twentieth more for the weights (7 TB/s) where the small-M kernel's workgroups of
// 16 columns fill whole rounds of the CUs?  Measured (us, streaming / small-M): 8192
// x 8192, M = 3 28.4 / 26.1, 8 28.6 / 30.2; 7168 x 2048, M = 12 11.7 / 10.4; 5120 x 1536, M
// = 16 8.8 / 7.9, 24 9.0 / 9.6; 4096 x 14336, M = 6 26.4 / 25.8, 8 26.4 / 27.3; 6144 x 4096
// (one and a half rounds), M = 6 14.5 / 15.6.  (Within 6 % of the better one
// elsewhere: 57344 x 8192, M = 3 164.5 / 159.7; 7168 x 2048, M = 24 12.6 / 11.9.)
static bool skinny_estimate(int64_t M, int64_t N, int64_t K, int splits) {
  const double weights_us = 2.0 * N * K / 7e6, rounds = (double)N / 16 / kNumCUs;
  const double idle_us = (std::ceil(rounds) / rounds - 1) * weights_us;
  return (double)M * N * K / 8 / 15e6 + idle_us <= (splits > 1 ? 2.5 : 0.0) + 0.05 * weights_us;
}

// One rule for the path of a linear, shared by the workspace query and the
// launch.  split_ok == false (no caller workspace) plans only paths that need
// none: the small-M kernel or unsplit tiles.
LinearPlan plan_linear(int64_t M, int64_t N, int64_t K, bool bf16, bool split_ok) {
  LinearPlan p{};
  if (!bf16) { p.path = LinearPlan::kF32; return p; }
  const int32_t force_tile = tuning(OPSCALE_TUNE_GEMM_TILE);
  const int32_t skinny = tuning(OPSCALE_TUNE_GEMM_SKINNY);
  p.path = LinearPlan::kTiled;
  // Decode batches of up to 128 rows: the weight-streaming kernel, its K split
  // (if any) through the workspace; or the small-M kernel, which reduces its
  // K split in LDS and needs no workspace, but reads all of x per 16 columns.
  // That extra x traffic (M N K / 8 bytes from L2) against the other's second
  // launch and partials, which grow with its K ranges, draws the line.
  // Measured (us, streaming / small-M kernel; splits in brackets): QKV 6144 x
  // 4096 [4] M = 4 14.7 / 14.4, M = 8 14.7 / 15.7; O 4096 x 4096 [8] M = 8 13.3 /
  // 9.6, M = 16 13.5 / 11.4, M = 32 13.9 / 15.2; down 4096 x 14336 [8] M = 4 27.6 /
  // 24.7, M = 8 27.4 / 27.4; gate-up 28672 x 4096 [1] M = 1 41.6 / 39.9, M = 4
  // 40.1 / 44.2, M = 16 40.4 / 64.5; 57344 x 8192 [1] M = 2 163 / 153, M = 4 equal.
  // Beyond 32 rows with K past 8192 the split-K tiles are as fast or faster (8192
  // x 28672 at M = 48 89.7 against 91.5); past 128 rows everywhere.
  const int32_t dec = tuning(OPSCALE_TUNE_GEMM_DECODE);
  LinearPlan d{};
  if (force_tile < 0 && dec != 0 && decode_linear_supported(M, N, K) && (dec == 1 || K <= 8192 || M <= 32)) {
    const int ds = tuning(OPSCALE_TUNE_GEMM_SPLITK) == 0 ? 1 : decode_linear_splits(M, N, K);
    if (ds <= 1 || split_ok) {
      d.path = LinearPlan::kDecode;
      d.splits = ds;
      d.ws_bytes = ds > 1 ? decode_linear_ws_bytes(M, N, K) : 0;
    }
  }
  const bool streamed = d.path == LinearPlan::kDecode;
  if (force_tile < 0 && skinny != 0 && !(streamed && dec == 1)) {
    const bool few = streamed ? M <= 2 || (double)M * N * K <= 3.5e7 * d.splits || skinny_estimate(M, N, K, d.splits)
                              : skinny_linear_preferred(M, N, K);
    if (skinny_linear_supported(M, N, K) && (skinny == 1 || few)) {
      p.path = LinearPlan::kSkinny;
      return p;
    }
  }
  if (streamed) return d;
  // Otherwise up to 128 rows split K over workgroups (fp32 partials in the
  // workspace, summed in split order by a second kernel) on tiles of 64 or 128
  // rows, so that the matrix cores work on little padding.
  if (force_tile < 0 && split_ok && tuning(OPSCALE_TUNE_GEMM_SPLITK) != 0 && M <= 128) {
    p.splits = M <= 64 ? splitk_count(64, 256, M, N, K) : splitk_count(128, 256, M, N, K);
    p.cfg = M <= 64 ? kCfgSk64 : kCfgSk128;
    if (p.splits > 1) {
      p.ws_bytes = split_bytes(M, N, K, p.splits);
      return p;
    }
    p.splits = 0;
  }
  // A last round at most half full runs split over K: 2-4 ranges per tile
  // (at most one workgroup per CU in all), each at least 8 slices long.
  const bool tail_ok = split_ok && tuning(OPSCALE_TUNE_GEMM_TAIL) != 0;
  auto tail_splits = [&](int64_t tiles) {
    const int64_t tail = tiles % kNumCUs;
    if (!tail_ok || tiles <= kNumCUs || tail == 0 || tail * 2 > kNumCUs) return 0;
    const int ts = (int)std::min<int64_t>(std::min<int64_t>(4, kNumCUs / tail), K / (8 * 64));
    return ts < 2 ? 0 : ts;
  };
  auto tiles_of = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  if (force_tile >= 0) {
    static constexpr struct { int bm, bn, cfg; } forced[] = {
        {256, 256, kCfgW4}, {192, 256, kCfgT192}, {256, 128, kCfgMid}, {256, 256, kCfgBig8}};
    const auto& f = forced[force_tile];
    p.cfg = f.cfg == kCfgW4 && N >= kW4MaxN ? kCfgBig8 : f.cfg;
    p.tail_splits = tail_splits(tiles_of(f.bm, f.bn));
    if (p.tail_splits > 1) p.ws_bytes = tail_bytes(f.bm, f.bn, M, N, K, p.tail_splits);
    return p;
  }
  // 256x256 or 128x256 tiles, whole or split over K (small M), whichever the
  // estimate below has faster.  One workgroup runs per CU; a launch takes full
  // rounds and a last one, a slice of K takes longer the more CUs run (power
  // and bandwidth shared), and a K split pays for its partials (written and
  // read) and a second launch.  Microseconds per slice fitted to measured
  // launches: 256x256 1.1 up to half the CUs, 1.34 on all (1500 x 6144 x 4096
  // 144 tiles 75 us, 3000 x 4096 x 4096 192 tiles 83, 4500 x 28672 x 4096 full
  // rounds); 128x256 0.70 to 0.86 (700 x 6144 144 tiles 50, 1500 x 4096 192 tiles
  // 53, 512 x 28672 full rounds).  (192x256 and 256x128 tiles of the older
  // kernels, 1.3 and 1.9 times the time per element, never win.)
  struct Tile { int bm, cfg; double busy, all, fixed; };
  static constexpr Tile kTiles[] = {{256, kCfgW4, 1.1, 1.34, 5.0}, {128, kCfgH4, 0.70, 0.86, 4.0}};
  double best = 0;
  for (const Tile& t : kTiles) {
    const int64_t tiles = tiles_of(t.bm, 256), slices = (K + 63) / 64;
    auto slice_us = [&](int64_t wgs) {
      const double u = (double)wgs / kNumCUs;
      return t.busy + std::max(0.0, u - 0.5) * 2 * (t.all - t.busy);
    };
    auto consider = [&](double us, int splits, int tail, size_t bytes) {
      if (best != 0 && us >= best) return;
      best = us;
      p.cfg = t.cfg == kCfgW4 && N >= kW4MaxN ? kCfgBig8 : t.cfg;
      p.splits = splits;
      p.tail_splits = tail;
      p.ws_bytes = bytes;
    };
    auto partials_us = [](double bytes) { return 3.0 + 2 * bytes / 7e6; };
    const int64_t full = tiles / kNumCUs, rem = tiles % kNumCUs;
    const int ts = t.cfg == kCfgW4 ? tail_splits(tiles) : 0;
    const size_t tail_b = ts > 1 ? tail_bytes(t.bm, 256, M, N, K, ts) : 0;
    double us = full * (slices * t.all) + t.fixed * (t.cfg == kCfgW4 ? 1 : full + (rem ? 1 : 0));
    if (rem) us += ts > 1 ? (double)slices / ts * t.all + partials_us((double)tail_b) : slices * slice_us(rem);
    consider(us, 0, ts, tail_b);
    const int sp = split_ok && tuning(OPSCALE_TUNE_GEMM_SPLITK) != 0 ? splitk_count(t.bm, 256, M, N, K) : 0;
    if (sp > 1) {
      const int ranges = split_ranges(K, sp, 64);
      const size_t b = split_bytes(M, N, K, sp);
      consider((double)(split_chunk(K, sp, 64) / 64) * slice_us(tiles * ranges) + t.fixed + partials_us((double)b), sp, 0,
               b);
    }
  }
  return p;
}

hipError_t launch_linear(const LinearPlan& p, const void* x, const void* W, const void* bias, void* y, int64_t M,
                         int64_t N, int64_t K, void* ws, hipStream_t s) {
  float* part = static_cast<float*>(ws);
  switch (p.path) {
    case LinearPlan::kSkinny:
      return launch_linear_skinny(x, W, bias, y, M, N, K, s);
    case LinearPlan::kDecode:
      return launch_linear_decode(x, W, bias, y, M, N, K, p.splits, ws, s);
    case LinearPlan::kTiled:
      switch (p.cfg) {
        case kCfgBig8: return launch_gemm_bf16<CfgBig8>(x, W, bias, y, M, N, K, s, p.splits, p.tail_splits, part);
        case kCfgH4: return launch_gemm_h4(x, W, bias, y, M, N, K, s, p.splits, part);
        case kCfgW4: return launch_gemm_w4(x, W, bias, y, M, N, K, s, p.splits, p.tail_splits, part);
        case kCfgT192: return launch_gemm_bf16<CfgT192>(x, W, bias, y, M, N, K, s, p.splits, p.tail_splits, part);
        case kCfgMid: return launch_gemm_bf16<CfgMid>(x, W, bias, y, M, N, K, s, p.splits, p.tail_splits, part);
        case kCfgSk64: return launch_gemm_bf16<CfgSk64>(x, W, bias, y, M, N, K, s, p.splits, p.tail_splits, part);
        default: return launch_gemm_bf16<CfgSk128>(x, W, bias, y, M, N, K, s, p.splits, p.tail_splits, part);
      }
    default: break;
  }
  return launch_linear_f32(x, W, bias, y, M, N, K, s);
}

}  // namespace opscale
