// How GEMM work items are dealt to workgroups and CUs.  Plain C++, so the schedule
// can be checked on the host.
#pragma once

#include <cmath>
#include <cstdint>

#ifdef __HIPCC__
#define OPS_HD __host__ __device__
#else
#define OPS_HD
#endif

namespace opscale {

constexpr int kNumCUs = 256;  // MI355X compute units

// Chains of the four-wave GEMM.
//
// A launch's items run in rounds of kNumCUs.  Workgroups come in groups of
// kNumCUs: group g takes a run of rounds, workgroup p of the group item p of
// each of them (a chain).  A chain is at most kMaxChain items and at most a
// third of the rounds that its group and the groups behind it hold, so the
// launch ends in single items and the workgroups that start late are the short
// ones: on any number of CUs (a CU-masked stream, or beside another kernel that
// holds some) the launch takes no longer than with one item per workgroup.
// Chains of four throughout doubled what they could not finish in one pass: the
// 2048-token gate-up on 90 % of the CUs took as long as on half of them.
constexpr int kMaxChain = 4;

// Rounds that a group takes of the `left` that remain.
OPS_HD inline int chain_length(int left) {
  const int third = left / 3;
  return third < 1 ? 1 : third > kMaxChain ? kMaxChain : third;
}

// Groups in front whose chains all have kMaxChain items.
OPS_HD inline int full_chains(int rounds) {
  return rounds < 3 * kMaxChain ? 0 : (rounds - 3 * kMaxChain) / kMaxChain + 1;
}

// First round and chain length of a group (length 0: past the last round).
struct Chain {
  int first, len;
};
OPS_HD inline Chain chain_of(int group, int rounds, bool chained) {
  if (!chained) return Chain{group, group < rounds ? 1 : 0};
  const int full = full_chains(rounds);
  if (group < full) return Chain{group * kMaxChain, kMaxChain};
  int first = full * kMaxChain, len = chain_length(rounds - first);
  for (int g = full; g < group && first < rounds; ++g) {
    first += len;
    len = chain_length(rounds - first);
  }
  return Chain{first, first < rounds ? len : 0};
}

// Workgroups of a launch of `items` items; if not `exact`, of a launch of any
// number up to that (the groups never grow fewer with the rounds, but their
// last one may have to be whole).
inline int64_t chain_grid(int64_t items, bool chained, bool exact) {
  const int rounds = (int)((items + kNumCUs - 1) / kNumCUs);
  int groups = rounds;
  if (chained) {
    groups = full_chains(rounds);
    for (int left = rounds - groups * kMaxChain; left > 0; left -= chain_length(left)) ++groups;
  }
  // (the last group's chains are single items)
  return exact ? (int64_t)(groups - 1) * kNumCUs + items - (int64_t)(rounds - 1) * kNumCUs : (int64_t)groups * kNumCUs;
}

// The mixture-of-experts GEMMs of decode batches, on tiles of 64 rows and 256 of N
// columns.
//
// Tiles of a launch: `rows` token-slot pairs over E experts, as if routed evenly (the
// host does not see the routing): experts that get a row, and a second tile for
// those that get more than 64 (binomial counts, taken as normal).
inline double grouped_tiles(int64_t rows, int64_t N, int64_t E) {
  const double used = E * (1.0 - std::pow(1.0 - 1.0 / E, (double)rows)), mean = rows / used;
  return used * (1.0 + 0.5 * std::erfc((64.5 - mean) / std::sqrt(2.0 * mean))) * (double)((N + 255) / 256);
}

// One workgroup of 160 KB per CU with three slices of K in flight, rather than
// two of 80 KB with one each?  Either way it is the weights that take the time.
// Alone on its CU the deep ring streams faster (up to 256 tiles, us, two / one per
// CU: 16 experts 6144 x 2688, 84 tiles 184 / 151; 8 experts of 14336, the 32 tiles
// of down 349 / 285), but it runs in rounds of 256 tiles where the pairs run in
// rounds of 512: a remainder of 257 to 511 is one round of pairs, its CUs
// sharing the bandwidth, and two of the others (294 tiles 289 / 331, 336 394 / 427,
// 800 473 / 503, 1372 761 / 766), one of up to 256 the reverse (672 563 / 530, 1160
// 586 / 561, 1280 645 / 629).  The same over 12 expert shapes of 1 to 512 tokens, K of
// 768 to 14336.  (Weights that fit the last-level cache, e.g. one expert called over and
// over, go 1-3 us the other way below 130 tiles, 18 at 8 tiles of K = 8192.)  On a
// share of the CUs the estimate is too coarse for the shorter rounds: pairs (64
// experts of 2560 on 64 CUs, 64 tokens 1337 / 1451, 256 tokens 1440 / 1517).
inline bool grouped_deep_ring(int64_t rows, int64_t N, int64_t E, int cus) {
  if (cus < kNumCUs) return false;
  const double last = std::fmod(std::round(grouped_tiles(rows, N, E)), 2.0 * kNumCUs);
  return last > 0 && last <= kNumCUs;
}

// The decode-batch linear on a stream of fewer CUs (a CU mask): the waves, of 16
// columns each, per workgroup that give a CU the fewest columns, K in `splits`
// ranges.  The shape for the whole chip is often exactly a workgroup per CU, which
// leaves some CUs two on any smaller share (us, 48 x 28672 x 4096 on 230 CUs, 256
// workgroups of seven waves 75, 224 of eight 46; on 192 74, 359 of five 59; 48 x
// 6144 x 4096 on 192, 256 of six 25.7, 192 of eight 19.4).  Workgroups are dealt
// evenly to the 32 shader engines, so a share counts as 32 times its whole CUs per
// engine (154 CUs, 299 workgroups: as 128 CUs, three on some).
constexpr int kMinStreamWaves = 5, kMaxStreamWaves = 8;
constexpr int kEngines = 32;
inline int stream_waves(int64_t N, int splits, int cus) {
  const int even = cus < kEngines ? cus : cus / kEngines * kEngines;
  int best = 0;
  int64_t best_cost = 0;
  for (int nw = kMaxStreamWaves; nw >= kMinStreamWaves; --nw) {
    const int64_t wgs = (N + 16 * nw - 1) / (16 * nw) * splits;
    const int64_t cost = (wgs + even - 1) / even * nw;
    if (best == 0 || cost < best_cost) best = nw, best_cost = cost;
  }
  return best;
}

}  // namespace opscale
