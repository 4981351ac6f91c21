// Host arithmetic of launches, apart from the kernels so that a plain C++ compiler can test it.
#ifndef MOE_LAUNCH_RULES_H
#define MOE_LAUNCH_RULES_H

#include <stdint.h>

namespace moe {

// HIP launches nothing with 2^32 threads or more in a grid dimension.
constexpr bool launch_fits(int64_t blocks, int threads) { return blocks * threads < (int64_t(1) << 32); }

constexpr int RT_TM = 16;              // token rows of an MFMA tile
constexpr int RT_THREADS = 512;        // threads of a routing block

// Tokens per block of moe_route's per-tile kernel, a power of two up to RT_TM; the other rows of the tile idle.
// cus: compute units.  Both types: no more blocks than a launch takes.
//
// bf16: the fewest that leave no more than one block per CU.  A block has a CU to itself (512 threads of more than 128
// registers), so blocks past the first round are a second one, which costs more than the shorter tail of every block
// saves.  At 256 CUs the tile is full from 2049 tokens on; from 4097 there is more than one block per CU.
// (Measured, the most tokens that still give 256 blocks -> this, us: d = 4096, E = 8, 257 tokens 13.4 -> 8.1, 500 13.8
// -> 8.0, 1000 14.6 -> 8.5, 1500 15.7 -> 10.2; d = 5120, E = 16, 1000 tokens 25.6 -> 14.5, 3000 30.9 -> 26.3; d = 4096,
// E = 256, 1500 tokens 136 -> 74, 4000 147 -> 89; nowhere slower at E = 8 to 256, d = 1048, 2048 and 4096, 64 to 4000
// tokens: the same at 512, 1024 and 2048.)
//
// fp32: every token takes the exact pass, in which the whole block works on one token after the other, so one token
// per block spreads a batch best.  More, the largest number that gives no CU more tokens (per(t) blocks of t tokens
// each, at most), where that saves something:
//   - small gates of up to 64 experts: the fixed part of a block, if the blocks of a CU come in pairs (one alone has
//     nobody to hide its waits).  d = 128, E = 16, 2000 tokens 21.3 -> 19.7 us, 8192 77 -> 68; from 24 KiB on two tokens
//     only (d = 1024, E = 16, 2000 tokens: one 26.0, two 25.1, four 27.3), from 64 KiB on one;
//   - more than 128 experts, whose LDS leaves room for one block on a CU: the fixed part again.  d = 128, E = 256, 8192
//     tokens 426 -> 405;
//   - gates of 512 KiB and more of 65 to 128 experts, if one block per CU is left: tokens that a CU takes one after the
//     other find more of the gate in its caches than the tokens of two blocks at once.  d = 1024, E = 128, 512 tokens
//     60 -> 52, 2048 205 -> 191; the same layer with d = 512 is slower so (1000 tokens 16 %).
// (Against the rule that gave every CU a block or more, as bf16 had: E = 4 to 256, d = 128 to 4096, 16 to 16384 tokens,
// 397 shapes: 0.97 to 1.76 times as fast.)
inline int route_tokens_per_block(bool bf16, int T, int E, int d, int cus) {
  auto blocks = [&](int tpb) { return (static_cast<int64_t>(T) + tpb - 1) / tpb; };
  int tpb = 1;
  if (bf16) {
    while (tpb < RT_TM && blocks(tpb) > cus) tpb <<= 1;
  } else {
    const int64_t gate = static_cast<int64_t>(E) * d * 4;
    auto per = [&](int t) { return (blocks(t) + cus - 1) / cus; };
    for (int t = 2; t <= RT_TM; t <<= 1) {
      if (per(t) * t > per(1)) continue;
      if (E > 128 || (E > 64 && gate >= 512 * 1024 && per(t) == 1) ||
          (E <= 64 && gate <= (t == 2 ? 64 : 24) * 1024 && per(t) % 2 == 0))
        tpb = t;
    }
  }
  while (tpb < RT_TM && !launch_fits(blocks(tpb), RT_THREADS)) tpb <<= 1;
  return tpb;
}

}  // namespace moe
#endif
