// Consumers of the expert-load statistic (Sections 3.3 and 4.2, Algorithm 1): the coefficient of
// variation of a layer's per-replica loads, the greedy Expert Scaling heuristic, and the even cut
// of each expert's row segment into its replicas' pieces.
//
// Algorithm 1 adds one replica per step to the expert whose replicas carry the largest load, until
// the CV of the per-replica loads is at most V or no further replica fits into the layer's memory
// cap.  The steps depend on each other, E is at most 256 and the data fits in registers, so ONE
// wave runs the whole loop: a lane owns experts lane, lane+64, ...; the straggler comes from a
// wave-wide arg-max (the paper's text uses a max-heap on the host; 64 lanes comparing at once
// replace it).  Bound by the chain of dependent instructions; scale_kernel takes the steps that no other can
// come between in one round of its loop.  Per-replica loads W_e / R_e are compared as fp64 quotients, which is exact: two
// different quotients with W < 2^31 and R <= 65537 < 2^17 differ by at least one part in
// W_a R_b < 2^48, more than a rounding (2^-53) can close, and equal ones round to the same
// number; equal loads go to the lowest expert index.  No host synchronisation: loads in,
// replica counts out, both on the device, so the counts that `moe_count_and_permute` (or a predictor's
// routing pass) has just produced can be consumed on the same stream.
#include <type_traits>

#include "moe_internal.h"

namespace moe {

// Wave-wide maximum / minimum of a 32-bit value by DPP (lane swaps in quads, half-row and row mirrors,
// two row broadcasts), read from lane 63.  ROWS = false: of lanes 0 .. 15 only (four steps).
template <bool MAX, bool ROWS = true> __device__ __forceinline__ uint32_t wave_extreme(uint32_t v) {
  auto step = [](uint32_t x, auto ctrl, auto rows) {
    const uint32_t o = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
        static_cast<int>(x), static_cast<int>(x), decltype(ctrl)::value, decltype(rows)::value, 0xF, false));
    return MAX ? max(x, o) : min(x, o);
  };
  using std::integral_constant;
  v = step(v, integral_constant<int, 0xB1>{}, integral_constant<int, 0xF>{});
  v = step(v, integral_constant<int, 0x4E>{}, integral_constant<int, 0xF>{});
  v = step(v, integral_constant<int, 0x141>{}, integral_constant<int, 0xF>{});
  v = step(v, integral_constant<int, 0x140>{}, integral_constant<int, 0xF>{});
  if constexpr (!ROWS) return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
  v = step(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});
  v = step(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 63));
}
__device__ __forceinline__ uint32_t hi32(double v) { return static_cast<uint32_t>(__double2hiint(v)); }
__device__ __forceinline__ uint32_t lo32(double v) { return static_cast<uint32_t>(__double2loint(v)); }
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum over the wave by DPP (prefix sums inside the rows of 16 lanes, two row broadcasts), read from lane 63.
// ROWS = false: of lanes 0 .. 15 only.
template <bool ROWS = true> __device__ __forceinline__ double wave_sum_dpp(double v) {
  auto step = [](double x, auto ctrl, auto rows) {
    return x + __hiloint2double(
        __builtin_amdgcn_update_dpp(0, __double2hiint(x), decltype(ctrl)::value, decltype(rows)::value, 0xF, false),
        __builtin_amdgcn_update_dpp(0, __double2loint(x), decltype(ctrl)::value, decltype(rows)::value, 0xF, false));
  };
  using std::integral_constant;
  v = step(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});
  v = step(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});
  v = step(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});
  v = step(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});
  if constexpr (!ROWS) return readlane_f64(v, 15);
  v = step(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});
  v = step(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});
  return readlane_f64(v, 63);
}

// The same in fp32.  ROWS = false: of lanes 0 .. 15 only.
template <bool ROWS> __device__ __forceinline__ float wave_sum_f32(float v) {
  auto step = [](float x, auto ctrl, auto rows) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, decltype(rows)::value,
                                                          0xF, decltype(rows)::value == 0xF));
  };
  using std::integral_constant;
  v = step(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});
  v = step(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});
  v = step(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});
  v = step(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});
  if constexpr (!ROWS) return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 15));
  v = step(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});
  v = step(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Q: experts per lane (E <= 64 Q).  One dependent chain per round of the loop, so a round takes as many steps as
// it can:
//   - an expert whose quotient W / R is above every expert's quotient after a further split, W / (R + 1), is
//     split before any expert is split twice: all such experts together are the next steps.  Their order matters only
//     where the budget ends among them (the largest first) and where CV may fall to V among them;
//   - CV is not recomputed: with S2 = sum W^2 / R it exceeds V exactly if n S2 > (1 + V^2) (sum W)^2.  S2 falls and n
//     grows with every step, so if (n + 1) times the S2 after the round is above (fp32 tells to 1e-4), it is above
//     after every step of it.  If that is not enough: a step lowers S2 by W/R * W/(R+1); with m the largest such
//     drop of the round, S2 after j of its c steps is at least S2 - j m, and (n + j) (S2 - j m) is least at j = 1
//     or j = c.  Where that does not settle it, the next SC_SINGLES steps (one, if no expert is above all further
//     splits) are taken one by one: the straggler by arg-max, S2 in fp64, summed once for these steps and lowered by each
//     step's drop (the error, below 1e-13, is far inside the 1e-9 within which the definition of CV decides, as it does
//     for the two values reported).  CV near V stays near V for a while, and each attempt at a whole round costs a step;
//   - the quotients after one and after two further splits are kept, so the division for the experts just split is
//     not needed in the next round.
// Bound by the chain of a round (DPP maxima and a DPP sum; SMALL: up to 16 experts, four DPP steps each instead of
// six).  Measured on Zipf loads, calls back to back, every step by itself -> rounds, one step where they fail -> now, us:
// 64 experts and 64 further replicas 20.2 -> 10.2 -> 9.2, 128 and 256 91 -> 33 -> 32, 256 and 1000 433 -> 144 -> 137;
// 8 and 30, V = 0 10.8 -> 11.8 -> 7.9, V = 0.1 10.8 -> 16.5 -> 8.9, V = 0.3 (4 steps) 4.4 -> 5.5 -> 3.9.
constexpr int SC_SINGLES = 16;
template <int Q, bool SMALL = false>
__global__ __launch_bounds__(MOE_WAVE) void scale_kernel(const int32_t* __restrict__ loads, int E,
                                                         int max_extra, double cv_threshold,
                                                         int32_t* __restrict__ replicas,
                                                         double* __restrict__ cv_out) {
  const int lane = lane_id();
  double w[Q], key[Q], next[Q], third[Q];      // W, W / R, W / (R + 1), W / (R + 2)
  int r[Q];
  long long s1 = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = lane + MOE_WAVE * q;
    const int load = e < E ? max(loads[e], 0) : 0;
    s1 += load;
    w[q] = key[q] = static_cast<double>(load);
    next[q] = 0.5 * w[q];
    third[q] = w[q] / 3.0;
    r[q] = 1;
  }
  // (exact: below 2^53)
  s1 = static_cast<long long>(wave_sum_dpp(static_cast<double>(s1)));
  int n = E;                                   // replicas in the layer
  int extra = 0;
  // CV of the multiset {W_e / R_e, R_e times}: population std / mean
  auto cv_exact = [&]() -> double {
    if (s1 <= 0) return 0.0;
    const double mean = static_cast<double>(s1) / static_cast<double>(n);
    double part = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (lane + MOE_WAVE * q < E) {
        const double dv = key[q] - mean;
        part += static_cast<double>(r[q]) * dv * dv;
      }
    }
    return readlane_f64(sqrt(wave_sum_dpp(part) / static_cast<double>(n)) / mean, 0);
  };
  const double cv_first = cv_exact();
  const double limit = (1.0 + cv_threshold * cv_threshold) * static_cast<double>(s1) * static_cast<double>(s1);
  const double surely_over = limit * (1.0 + 1e-9), surely_under = limit * (1.0 - 1e-9);
  const float over_f32 = static_cast<float>(limit) * 1.0001f;
  bool more = max_extra > 0 && cv_first > cv_threshold;
  while (more) {                               // wave-uniform
    uint32_t mn = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) mn = max(mn, hi32(next[q]));
    const uint32_t top_next = wave_extreme<true, !SMALL>(mn);
    // (upper words of the non-negative doubles: equal ones wait for a later round)
    bool take[Q];
    int count = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      take[q] = hi32(key[q]) > top_next;
      count += __popcll(__ballot(take[q]));
    }
    if (count > max_extra - extra) {           // only the largest fit the budget
      const int left = max_extra - extra;
      int rank[Q] = {};
#pragma unroll
      for (int p = 0; p < Q; ++p)
        for (unsigned long long m = __ballot(take[p]); m != 0ull; m &= m - 1) {
          const int l = __ffsll(static_cast<long long>(m)) - 1;
          const double k = readlane_f64(key[p], l);
          const int e = l + MOE_WAVE * p;
#pragma unroll
          for (int q = 0; q < Q; ++q) rank[q] += k > key[q] || (k == key[q] && e < lane + MOE_WAVE * q) ? 1 : 0;
        }
#pragma unroll
      for (int q = 0; q < Q; ++q) take[q] = take[q] && rank[q] < left;
      count = left;
    }
    float part_f = 0.f;                        // S2 after the round
#pragma unroll
    for (int q = 0; q < Q; ++q) part_f += static_cast<float>(w[q]) * static_cast<float>(take[q] ? next[q] : key[q]);
    const float s2f = wave_sum_f32<!SMALL>(part_f);
    bool over = cv_threshold < 0.0 || static_cast<float>(n + 1) * s2f > over_f32;
    if (!over && count > 1) {
      float drop = 0.f, all = 0.f;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float d = take[q] ? static_cast<float>(key[q]) * static_cast<float>(next[q]) : 0.f;
        drop = fmaxf(drop, d);
        all += d;
      }
      const float before = s2f + wave_sum_f32<!SMALL>(all);
      drop = __uint_as_float(wave_extreme<true, !SMALL>(__float_as_uint(drop)));   // (not negative: ordered as integers)
      over = fminf(static_cast<float>(n + 1) * (before - drop),
                   static_cast<float>(n + count) * (before - static_cast<float>(count) * drop)) > over_f32;
    }
    int singles = count == 0 ? 1 : over ? 0 : SC_SINGLES;      // steps to be taken one by one
    if (singles == 0) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (take[q]) {
          key[q] = next[q];
          next[q] = third[q];
          r[q] += 1;
        }
        third[q] = w[q] / static_cast<double>(r[q] + 2);
      }
      n += count;
      extra += count;
      more = extra < max_extra;
      continue;
    }
    double part = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) part += w[q] * key[q];
    double s2 = wave_sum_dpp<!SMALL>(part);
    for (; singles > 0 && more; --singles) {
      // the straggler: largest quotient, lowest index
      uint32_t mk = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) mk = max(mk, hi32(key[q]));
      const uint32_t top = wave_extreme<true, !SMALL>(mk);
      if (top == 0u) {                         // every load is zero: nothing to split
        more = false;
        break;
      }
      unsigned long long who[Q];
      int tied = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        who[q] = __ballot(hi32(key[q]) == top);
        tied += __popcll(who[q]);
      }
      if (tied > 1) {
        uint32_t ml = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) ml = max(ml, hi32(key[q]) == top ? lo32(key[q]) : 0u);
        const uint32_t top_lo = wave_extreme<true, !SMALL>(ml);
#pragma unroll
        for (int q = 0; q < Q; ++q) who[q] = __ballot(hi32(key[q]) == top && lo32(key[q]) == top_lo);
      }
      bool found = false;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (!found && who[q] != 0ull) {        // uniform
          found = true;
          const int l = __ffsll(static_cast<long long>(who[q])) - 1;
          s2 -= readlane_f64(key[q] * next[q], l);
          if (lane == l) {
            key[q] = next[q];
            next[q] = third[q];
            r[q] += 1;
          }
          third[q] = w[q] / static_cast<double>(r[q] + 2);
        }
      }
      n += 1;
      extra += 1;
      if (cv_threshold >= 0.0) {
        const double lhs = static_cast<double>(n) * s2;
        more = lhs > surely_over;
        if (!more && !(lhs < surely_under)) more = cv_exact() > cv_threshold;
      }
      more = more && extra < max_extra;
    }
  }
  const double cv = extra > 0 ? cv_exact() : cv_first;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = lane + MOE_WAVE * q;
    if (e < E) replicas[e] = r[q];
  }
  if (cv_out && lane == 0) {
    cv_out[0] = cv_first;
    cv_out[1] = cv;
  }
}

// Exclusive prefix sum over the block's 256 threads of values below 2^31; *total = the sum.  By DPP on the
// halves of the values, whose sums over a wave fit 32 bits.  part: LDS, four entries (a caller that uses it twice
// passes two arrays).
__device__ __forceinline__ long long block_prefix(int v, long long* part, long long* total) {
  const int wave = threadIdx.x / MOE_WAVE;
  const long long incl = wave_scan_add(v & 0xFFFF) + (static_cast<long long>(wave_scan_add(v >> 16)) << 16);
  if (lane_id() == MOE_WAVE - 1) part[wave] = incl;
  __syncthreads();
  long long before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i < wave) before += part[i];
    all += part[i];
  }
  *total = all;
  return before + incl - v;
}
__device__ __forceinline__ int saturate31(long long v) { return static_cast<int>(min(v, 0x7FFFFFFFll)); }

// One block.  prefix[e] = number of segments before expert e (thread e computes it: a serial prefix by
// one thread took a trip to memory per expert); thread s-strided over the segments.
static_assert(MOE_MAX_E == 256, "one thread per expert");
__global__ __launch_bounds__(256) void segments_kernel(const int32_t* __restrict__ offsets,
                                                       const int32_t* __restrict__ replicas, int E,
                                                       int max_segments,
                                                       int32_t* __restrict__ seg_offsets,
                                                       int32_t* __restrict__ seg_expert,
                                                       int32_t* __restrict__ n_segments) {
  __shared__ int prefix[MOE_MAX_E + 1];
  __shared__ int rep[MOE_MAX_E], off[MOE_MAX_E + 1];
  __shared__ long long part[4];
  const int tid = threadIdx.x;
  const int mine = tid < E ? max(replicas[tid], 1) : 0;
  rep[tid] = mine;
  if (tid <= E) off[tid] = offsets[tid];
  if (tid == 0 && E == 256) off[256] = offsets[256];
  long long all;
  const long long before = block_prefix(mine, part, &all);
  if (tid < E) prefix[tid] = saturate31(before);
  if (tid == 0) {
    prefix[E] = saturate31(all);
    *n_segments = saturate31(all);
    seg_offsets[0] = offsets[0];
  }
  __syncthreads();
  const int total = min(prefix[E], max_segments);
  for (int s = tid; s < total; s += 256) {
    int lo = 0, hi = E - 1;                    // last expert whose prefix is <= s
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (prefix[mid] <= s) lo = mid; else hi = mid - 1;
    }
    const int e = lo;
    const long long R = rep[e];
    const long long c = max(off[e + 1] - off[e], 0);
    const long long rr = s - prefix[e];
    seg_expert[s] = e;
    seg_offsets[s + 1] = off[e] + static_cast<int32_t>((c * (rr + 1)) / R);
  }
}

}  // namespace moe

extern "C" int moe_scale_replicas(int32_t E, const int32_t* loads, int64_t expert_mem,
                                  int64_t mem_cap, double cv_threshold, int32_t* replicas,
                                  double* cv_out, void* hip_stream) {
  if (E < 1 || !loads || !replicas || expert_mem < 1 || mem_cap < 0) return MOE_ERR_INVALID_ARG;
  if (!(cv_threshold == cv_threshold)) return MOE_ERR_INVALID_ARG;   // NaN
  if (E > MOE_MAX_E) return MOE_ERR_UNSUPPORTED;
  const int64_t max_extra = mem_cap / expert_mem;
  if (max_extra > MOE_MAX_EXTRA_REPLICAS) return MOE_ERR_UNSUPPORTED;
  const auto kernel = E <= 16 ? moe::scale_kernel<1, true> : E <= 64 ? moe::scale_kernel<1> : E <= 128 ? moe::scale_kernel<2> : moe::scale_kernel<4>;
  hipLaunchKernelGGL(kernel, dim3(1), dim3(MOE_WAVE), 0, static_cast<hipStream_t>(hip_stream), loads, E,
                     static_cast<int>(max_extra), cv_threshold, replicas, cv_out);
  return moe::launch_status();
}

extern "C" int moe_replica_segments(int32_t E, const int32_t* offsets, const int32_t* replicas,
                                    int32_t max_segments, int32_t* seg_offsets,
                                    int32_t* seg_expert, int32_t* n_segments, void* hip_stream) {
  if (E < 1 || !offsets || !replicas || !seg_offsets || !seg_expert || !n_segments ||
      max_segments < 0)
    return MOE_ERR_INVALID_ARG;
  if (E > MOE_MAX_E) return MOE_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(moe::segments_kernel, dim3(1), dim3(256), 0,
                     static_cast<hipStream_t>(hip_stream), offsets, replicas, E, max_segments,
                     seg_offsets, seg_expert, n_segments);
  return moe::launch_status();
}

// ---------------------------------------------------------------------------------------------
// Expert Placement (Algorithm 2, Section 4.3): replicas from the most to the least loaded; a
// replica that is still alive where the previous round put it stays there, any other joins the
// GPU with the smallest aggregated load.  GPU loads are fp64 sums in placement order, and a step
// needs the loads that the steps before left: ONE wave runs the steps, lane g holding GPU g's load,
// count and slots.  Everything a step needs that does not depend on the loads is prepared by the whole
// block, PL_CHUNK steps at a time, in LDS: the order of the experts (all replicas of an expert carry
// W_e / R_e, so they are placed one after the other; ranks by counting, quotients compared exactly
// as in scale_kernel), and per step the load, the warm GPU and the place of the result.  Bound by
// the chain of dependent instructions from step to step:
//   - a run of warm steps is one fp64 addition each, in the lane of its GPU;
//   - a run of others, each to the shortest queue: an arg-min over the lanes (upper words of the non-negative doubles by
//     DPP, a ballot, lower words only on a tie);
//   - 64 steps in which a GPU may run out of slots: the same step by step, over the lanes with a free slot.
// Measured, calls back to back, every step looked up by itself -> now, us: 64 experts, 128 replicas, 8 GPUs, all warm
// 19.0 -> 7.1, 30 % new 22.5 -> 17.0, all new 31.5 -> 23.2; 256 experts, 1256 replicas, 8 GPUs 143 -> 42, 179 -> 137 and
// 270 -> 204; 40 GPUs, 128 replicas, all new 38.4 -> 28.6; slots that run out 32 -> 31.  (Lanes kept in the order of
// their loads, so that a run of new replicas needs no arg-min: a step is no shorter, and sorting them for each run
// cost 1.5 us on 16 GPUs.)
// ---------------------------------------------------------------------------------------------
namespace moe {

constexpr int PL_MAX_GPUS = MOE_WAVE;
constexpr int PL_CHUNK = 1024;
struct PlaceStep {
  double w;        // load of the replica
  int warm;        // GPU of the previous round, -1 = none
  int out;         // index of the replica in gpu_of
};

// WIDE: more than 16 GPUs.
template <bool WIDE>
__global__ __launch_bounds__(256) void place_kernel(
    const int32_t* __restrict__ loads, const int32_t* __restrict__ replicas, int E, int G,
    const int32_t* __restrict__ prev_replicas, const int32_t* __restrict__ prev_gpu,
    const int32_t* __restrict__ gpu_slots, int max_segments, int step_budget,
    int32_t* __restrict__ gpu_of, double* __restrict__ gpu_load, int32_t* __restrict__ gpu_count,
    int32_t* __restrict__ n_warm) {
  __shared__ __align__(16) PlaceStep step[PL_CHUNK + 1];   // (one more: the read ahead of the last step)
  __shared__ unsigned long long cold[PL_CHUNK / MOE_WAVE];    // steps without a warm GPU
  __shared__ double key[MOE_MAX_E];
  __shared__ int seg_start[MOE_MAX_E], prev_n[MOE_MAX_E], rep[MOE_MAX_E], rank[MOE_MAX_E];
  __shared__ long long prev_start[MOE_MAX_E];    // (the previous round's counts are the caller's: their sum may pass 2^31)
  __shared__ int order[MOE_MAX_E], order_start[MOE_MAX_E + 1];
  __shared__ long long part[3][4];
  const int tid = threadIdx.x, lane = lane_id();
  // thread e: expert e
  const int my_r = tid < E ? min(max(replicas[tid], 1), MOE_MAX_EXTRA_REPLICAS + 1) : 0;
  const int my_p = tid < E && prev_replicas ? max(prev_replicas[tid], 0) : 0;
  key[tid] = tid < E ? static_cast<double>(max(loads[tid], 0)) / static_cast<double>(my_r) : -1.0;
  long long total, dummy;
  seg_start[tid] = static_cast<int>(block_prefix(my_r, part[0], &total));    // (at most 256 * 65537)
  prev_start[tid] = block_prefix(my_p, part[1], &dummy);
  prev_n[tid] = my_p;
  rep[tid] = my_r;
  rank[tid] = 0;
  __syncthreads();
  {
    // rank: experts before this one, more loaded, or equal and lower.  `parts` threads per expert take a share
    // of the others each.
    const int per = E <= 64 ? 64 : E <= 128 ? 128 : 256, parts = 256 / per;
    const int e = tid & (per - 1), share = (E + parts - 1) / parts;
    const int first = tid / per * share, last = min(first + share, E);
    const double mine = key[e];
    int before = 0;
#pragma unroll 8
    for (int o = first; o < last; ++o) before += (key[o] > mine || (key[o] == mine && o < e)) ? 1 : 0;
    if (e < E && before) atomicAdd(&rank[e], before);
  }
  __syncthreads();
  if (tid < E) order[rank[tid]] = tid;
  __syncthreads();
  const int my_o = tid < E ? order[tid] : 0;
  order_start[tid] = static_cast<int>(block_prefix(tid < E ? rep[my_o] : 0, part[2], &dummy));
  if (tid == 0) order_start[MOE_MAX_E] = static_cast<int>(total);
  __syncthreads();
  const int steps = static_cast<int>(min(total, static_cast<long long>(step_budget)));

  double gload = 0.0;                          // lane g: GPU g
  int gcount = 0;
  const int gslots = (lane < G) ? (gpu_slots ? max(gpu_slots[lane], 0) : 0x7FFFFFFF) : 0;
  int warm = 0;
  // the GPU with the smallest load among those of `room` (lowest index on a tie), -1 if there is none
  auto shortest = [&](unsigned long long room) -> int {
    const bool free_slot = (room >> lane) & 1ull;
    const uint32_t h = free_slot ? hi32(gload) : 0xFFFFFFFFu;
    const uint32_t least = wave_extreme<false, WIDE>(h);
    if (least == 0xFFFFFFFFu) return -1;
    unsigned long long who = __ballot(h == least);
    if (__popcll(who) > 1) {
      const uint32_t l = h == least ? lo32(gload) : 0xFFFFFFFFu;
      const uint32_t least_lo = wave_extreme<false, WIDE>(l);
      who = __ballot(h == least && l == least_lo);
    }
    return __ffsll(static_cast<long long>(who)) - 1;
  };
  auto put = [&](double load, int g) {
    gload += lane == g ? load : 0.0;           // (loads are not negative: the other lanes keep their bits)
    gcount += lane == g ? 1 : 0;
  };
  for (int first = 0; first < steps; first += PL_CHUNK) {
    const int n = min(PL_CHUNK, steps - first);
    for (int base = 0; base < n; base += 256) {
      const int i = base + tid;
      int g = -1;
      if (i < n) {
        const int s = first + i;
        int lo = 0, hi = E - 1;                // last rank whose first step is <= s
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (order_start[mid] <= s) lo = mid; else hi = mid - 1;
        }
        const int e = order[lo], q = s - order_start[lo];
        if (q < prev_n[e]) g = prev_gpu[prev_start[e] + q];
        if (g < 0 || g >= G) g = -1;
        step[i].w = key[e];
        step[i].warm = g;
        step[i].out = seg_start[e] + q;
      }
      const unsigned long long c = __ballot(i < n && g < 0);
      if (lane == 0) cold[i / MOE_WAVE] = c;
    }
    __syncthreads();
    if (tid < MOE_WAVE) {
      for (int base = 0; base < n; base += MOE_WAVE) {
        const int cnt = min(MOE_WAVE, n - base);
        PlaceStep* const st = step + base;
        if (__ballot(lane < G && gcount > gslots - cnt) != 0ull) {   // a GPU may run out of slots
          unsigned long long room = __ballot(gcount < gslots);
          PlaceStep cur = st[0];
          for (int i = 0; i < cnt; ++i) {
            const PlaceStep next = st[i + 1];  // (past the block's last step: read, not used)
            const int wg = __builtin_amdgcn_readfirstlane(cur.warm);
            int g = wg;
            if (wg >= 0 && ((room >> wg) & 1ull)) ++warm;
            else g = shortest(room);
            if (lane == g) {
              gload += cur.w;
              gcount += 1;
            }
            room = __ballot(gcount < gslots);
            if (lane == 0) st[i].warm = g;     // the step's result, in place of its input
            cur = next;
          }
          continue;
        }
        const unsigned long long all = ~0ull >> (MOE_WAVE - G);
        const uint32_t c_lo = __builtin_amdgcn_readfirstlane(static_cast<int>(cold[base / MOE_WAVE]));
        const uint32_t c_hi = __builtin_amdgcn_readfirstlane(static_cast<int>(cold[base / MOE_WAVE] >> 32));
        const unsigned long long mask = static_cast<unsigned long long>(c_hi) << 32 | c_lo;
        int i = 0;
        while (i < cnt) {                      // wave-uniform
          const unsigned long long ahead = mask >> i;
          const int end = ahead == 0ull ? cnt : i + __ffsll(static_cast<long long>(ahead)) - 1;
          warm += end - i;
#pragma unroll 8
          for (; i < end; ++i) put(st[i].w, st[i].warm);
          if (i >= cnt) break;
          const unsigned long long again = ~(mask >> i);        // (not zero: bit 63 - i and above, or i = 0 and all cold)
          const int run = min(cnt - i, again == 0ull ? MOE_WAVE : __ffsll(static_cast<long long>(again)) - 1);
          double load = st[i].w;
          for (int t = 0; t < run; ++t) {
            const double next = st[i + t + 1].w;
            const int g = shortest(all);
            if (lane == g) {
              gload += load;
              gcount += 1;
            }
            if (lane == 0) st[i + t].warm = g;
            load = next;
          }
          i += run;
        }
      }
    }
    __syncthreads();
    for (int i = tid; i < n; i += 256)
      if (step[i].out < max_segments) gpu_of[step[i].out] = step[i].warm;
    __syncthreads();
  }
  if (tid < G) {
    gpu_load[tid] = gload;
    gpu_count[tid] = gcount;
  }
  if (tid == 0) *n_warm = warm;
}

}  // namespace moe

extern "C" int moe_place_replicas(int32_t E, const int32_t* loads, const int32_t* replicas,
                                  int32_t n_gpus, const int32_t* prev_replicas,
                                  const int32_t* prev_gpu, const int32_t* gpu_slots,
                                  int32_t max_segments, int32_t* gpu_of, double* gpu_load,
                                  int32_t* gpu_count, int32_t* n_warm, void* hip_stream) {
  if (E < 1 || n_gpus < 1 || !loads || !replicas || !gpu_of || !gpu_load || !gpu_count || !n_warm ||
      max_segments < 0)
    return MOE_ERR_INVALID_ARG;
  if ((prev_replicas == nullptr) != (prev_gpu == nullptr)) return MOE_ERR_INVALID_ARG;
  if (E > MOE_MAX_E || n_gpus > moe::PL_MAX_GPUS) return MOE_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(n_gpus <= 16 ? moe::place_kernel<false> : moe::place_kernel<true>, dim3(1), dim3(256), 0,
                     static_cast<hipStream_t>(hip_stream), loads, replicas, E, n_gpus, prev_replicas,
                     prev_gpu, gpu_slots, max_segments, E + MOE_MAX_EXTRA_REPLICAS, gpu_of, gpu_load,
                     gpu_count, n_warm);
  return moe::launch_status();
}
