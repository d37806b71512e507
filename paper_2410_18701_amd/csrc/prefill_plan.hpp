// Which kernel a step's bf16 prompts take, from the sizes alone.  Host code
// without a GPU header, so that the rule can be evaluated on its own.
#pragma once

#include <algorithm>
#include <cstdint>

namespace baton {

// Whether the kernel of 128 positions per workgroup and 32 per wave
// (prefill_fa32_kernel) is faster than the one of 64: `wgs` workgroups of 128
// positions over prompts of plen[0 .. n) tokens.  Its chain
// of blocks is 1.35 times as long in time, so it loses where the chains and not
// the matrix operations bound the launch: below one to two workgroups per CU
// (four run at head_dim 64 of the other kernel), with several long prompts a little
// later (a later prompt's longest tiles start after the first prompt's last), and
// with short prompts.  us per layer, 64 / 128 positions:
//  * head_dim 128, one prompt: 2 heads of 8192 tokens (128 workgroups) 120 / 161,
//    8 of 4096 (256) 71 / 90, 12 of 4096 (384) 87 / 97, 10 of 6000 (470) 151 / 142,
//    32 of 2048 (512) 64 / 61, 64 of 4096 (2048) 382 / 308; two prompts of 2048:
//    12 heads (384) 50 / 60, 16 (512) 64 / 73, 24 (768) 96 / 83; three of 3000, 8
//    heads (576) 100 / 90; two of 1024, 32 heads (512) 44 / 45;
//  * head_dim 64, one prompt: 4 heads of 8192 (256) 85 / 113, 10 of 6000 (470) 89 /
//    94, 16 of 4096 (512) 68 / 69, 32 of 4096 (1024) 123 / 103; two of 6000: 6 heads
//    (564) 103 / 122, 8 (752) 134 / 126; three of 3000, 10 heads (720) 76 / 86; four
//    of 1024, 32 heads (1024) 49 / 52, the product of workgroups and tokens half of
//    what the rule asks.
inline bool prefill_long(int32_t head_dim, const int32_t* plen, int32_t n, int64_t wgs) {
  int32_t longest = 0, n_long = 0;   // prompts over a quarter of the longest
  for (int32_t i = 0; i < n; ++i) longest = std::max(longest, plen[i]);
  for (int32_t i = 0; i < n; ++i) n_long += plen[i] > longest / 4;
  if (longest < 512 || longest * wgs < (head_dim == 64 ? 1 << 21 : 1 << 20)) return false;
  return wgs >= (head_dim == 64 ? (n_long == 1 ? 512 : 750) : (n_long == 1 ? 470 : 520));
}

}  // namespace baton
