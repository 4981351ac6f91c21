// Host arithmetic of launches, apart from the kernels so that a plain C++ compiler can test it.
#ifndef MOE_LAUNCH_RULES_H
#define MOE_LAUNCH_RULES_H

#include <stdint.h>

namespace moe {

// HIP launches nothing with 2^32 threads or more in a grid dimension.
constexpr bool launch_fits(int64_t blocks, int threads) { return blocks * threads < (int64_t(1) << 32); }

constexpr int RT_TM = 16;              // token rows of an MFMA tile
constexpr int RT_THREADS = 512;        // threads of a routing block

// Tokens per block of moe_route's per-tile kernel, a power of two up to RT_TM (why these: launch_route).
inline int route_tokens_per_block(bool bf16, int T) {
  constexpr int CUS = 256;
  auto blocks = [&](int tpb) { return (static_cast<int64_t>(T) + tpb - 1) / tpb; };
  int tpb = 1;
  while (tpb < RT_TM && (bf16 ? blocks(tpb) > CUS : !launch_fits(blocks(tpb), RT_THREADS))) tpb <<= 1;
  return tpb;
}

}  // namespace moe
#endif
