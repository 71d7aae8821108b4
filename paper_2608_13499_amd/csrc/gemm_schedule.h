// How GEMM work items are dealt to workgroups and CUs.  Plain C++, so the schedule
// can be checked on the host.
#pragma once

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

}  // namespace opscale
