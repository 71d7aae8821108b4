// Which kernels a fp32 prefill attention call takes, and their launches.  Plain
// C++, so that it can be checked on the host.
#pragma once

#include <algorithm>
#include <cstdint>

#include "grid.h"

namespace opscale {

struct AttnF32Plan {
  int32_t row_len;  // prompts of up to this many tokens take a wave per (token, head); 0: none
  int64_t items;    // (tile, head) items of the others; 0: no such launch
  int32_t levels;   // > 0: `levels` tiles for every prompt; 0: a list of the tiles there are
  uint32_t grid;    // workgroups that go through the items
};

// cu_seqlens is on the device: the choice uses what the call states, B prompts of
// total_tokens in all, none longer than max_seqlen (an upper bound, maybe a
// loose one).
//
// A 32-query tile takes its time whatever it holds (7 us for the first 512 of
// heads of 64, 10.5 us for the first 256 of heads of 128; 9 and 28 ns each past
// them); a wave per (token, head) takes 5 us and 0.5 to 2 ns (64) or 1.2 to 4 ns
// (128) a token and head, growing with its keys.  Measured (us, wave / tile; heads x
// width, prompts): 4x64 1x48 5.9 / 7.4, 1x80 8.3 / 7.6; 32x64 1x33 6.2 / 7.5, 1x48 7.5 /
// 7.5; 8x128 1x33 7.1 / 10.6, 1x64 10.1 / 11.1, 1x96 13.9 / 11.9; 32x128 1x33 8.7 / 10.7,
// 1x64 16.2 / 11.5; 32x64 100x5 16 / 35, 64x10 21 / 24, 64x24 58 / 26; 32x128 100x5 26 /
// 104, 64x10 35 / 71, 64x24 101 / 73.
//
// A launch of `levels` tiles for every prompt needs no search (256x30, 4x64: 14.8
// against 19.0 from the list), but its tiles past a prompt's end cost about 31
// ns each (heads of 128; one prompt of 1000 and 500 of one token, 32 heads: 16
// ms, from the list 0.71, with the short ones a wave each 0.18; 512, 17, 100
// and 300 tokens 122 / 71 us).  (Where the bound alone hides that all are short,
// the list's empty launch costs 2-6 us: 100x5 under a bound of 2500, 8x128 9.9 ->
// 12.2.)
inline AttnF32Plan attn_f32_plan(int64_t B, int64_t total_tokens, int64_t max_seqlen, int64_t Hq, int64_t D) {
  const int64_t longest = std::min(max_seqlen, total_tokens), heads = total_tokens * Hq;
  AttnF32Plan p{};
  if (total_tokens <= kMaxGrid64 &&
      ((longest <= 64 && heads <= 1400) || longest <= (D > 64 ? 16 : 10))) {
    p.row_len = INT32_MAX;
    return p;
  }
  const int64_t slots = total_tokens / 32 + B;  // at least the tiles there are
  const int64_t levels = (longest + 31) / 32;
  if (B * levels <= slots + slots / 4) {
    p.levels = (int32_t)levels;
    p.items = B * levels * Hq;
  } else {
    // mostly short prompts: those take a wave each
    if (total_tokens <= kMaxGrid64 && total_tokens <= 16 * B) p.row_len = 32;
    p.items = (total_tokens / 32 + std::min(B, total_tokens / (p.row_len + 1))) * Hq;
  }
  p.grid = (uint32_t)std::min(p.items, kMaxGrid256);
  return p;
}

}  // namespace opscale
