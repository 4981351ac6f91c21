// Consumers of the expert-load statistic (Sections 3.3 and 4.2, Algorithm 1): the coefficient of
// variation of a layer's per-replica loads, the greedy Expert Scaling heuristic, and the even cut
// of each expert's row segment into its replicas' pieces.
//
// Algorithm 1 adds one replica per step to the expert whose replicas carry the largest load, until
// the CV of the per-replica loads is at most V or no further replica fits into the layer's memory
// cap.  The steps depend on each other, E is at most 256 and the data fits in registers, so ONE
// wave runs the whole loop: a lane owns experts lane, lane+64, ...; the straggler comes from a
// wave-wide arg-max (the paper's text uses a max-heap on the host; 64 lanes comparing at once
// replace it).  Bound by the chain of dependent instructions of a step; see scale_kernel for how
// it is kept short.  Per-replica loads W_e / R_e are compared as fp64 quotients, which is exact: two
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

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Q: experts per lane (E <= 64 Q).  What a step costs is its dependent chain, so
//   - the straggler is the largest fp64 quotient: a DPP maximum over the upper words of the (non-
//     negative) doubles, a ballot on equality, and a second pass over the lower words only when
//     more than one expert shares the upper one;
//   - the quotient after a further split, W / (R + 1), is kept beside the current one; the division
//     for the expert just split is issued at the head of the next step, beside that step's arg-max,
//     which does not need it;
//   - CV is not recomputed: with S2 = sum W^2 / R it exceeds V exactly if n S2 > (1 + V^2) (sum W)^2, and
//     a split changes S2 by W/R * W/(R+1).  Where that test is closer than 1e-9 (the increments' error
//     is below 1e-11: S2 is summed afresh every 256 steps, over which it shrinks at most 256-fold), the
//     definition decides, as it does for the two values reported.
// Measured: 64 experts, 64 further replicas 80 us with CV by its definition and an arg-max by 64-bit
// cross products over lane shuffles in every step, now 20 us.
constexpr int SC_REFRESH = 256;
template <int Q>
__global__ __launch_bounds__(MOE_WAVE) void scale_kernel(const int32_t* __restrict__ loads, int E,
                                                         int max_extra, double cv_threshold,
                                                         int32_t* __restrict__ replicas,
                                                         double* __restrict__ cv_out) {
  const int lane = lane_id();
  double w[Q], key[Q], next[Q];                // W, W / R, W / (R + 1)
  int r[Q];
  long long s1 = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = lane + MOE_WAVE * q;
    const int load = e < E ? max(loads[e], 0) : 0;
    s1 += load;
    w[q] = key[q] = static_cast<double>(load);
    next[q] = 0.5 * w[q];
    r[q] = 1;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s1 += __shfl_xor(s1, off);
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
    return readlane_f64(sqrt(wave_sum_f64(part) / static_cast<double>(n)) / mean, 0);
  };
  auto sum_w2_over_r = [&]() -> double {
    double part = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) part += w[q] * key[q];
    return readlane_f64(wave_sum_f64(part), 0);
  };
  const double cv_first = cv_exact();
  double s2 = sum_w2_over_r();
  const double limit = (1.0 + cv_threshold * cv_threshold) * static_cast<double>(s1) * static_cast<double>(s1);
  const double surely_over = limit * (1.0 + 1e-9), surely_under = limit * (1.0 - 1e-9);
  bool more = max_extra > 0 && cv_first > cv_threshold;
  int last = -1, last_q = 0;                   // the expert split in the step before: lane and slot
  double last_w = 0.0;
  int last_r = 1;
  while (more) {                               // wave-uniform
    const double pending = last_w / static_cast<double>(last_r + 1);
    uint32_t m = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) m = max(m, hi32(key[q]));
    const uint32_t top = wave_extreme<true>(m);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (lane == last && q == last_q) next[q] = pending;
    if (top == 0u) break;                      // every load is zero: nothing to split
    unsigned long long who[Q];
    int count = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      who[q] = __ballot(hi32(key[q]) == top);
      count += __popcll(who[q]);
    }
    if (count > 1) {
      uint32_t ml = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) ml = max(ml, hi32(key[q]) == top ? lo32(key[q]) : 0u);
      const uint32_t top_lo = wave_extreme<true>(ml);
#pragma unroll
      for (int q = 0; q < Q; ++q) who[q] = __ballot(hi32(key[q]) == top && lo32(key[q]) == top_lo);
    }
    int qs = Q - 1;                            // lowest index: lowest slot, then lowest lane
#pragma unroll
    for (int q = Q - 2; q >= 0; --q)
      if (who[q] != 0ull) qs = q;
    double drop = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (q == qs) {                           // uniform
        last = __ffsll(static_cast<long long>(who[q])) - 1;
        last_q = q;
        drop = readlane_f64(key[q] * next[q], last);
        last_w = readlane_f64(w[q], last);
        last_r = __builtin_amdgcn_readlane(r[q], last) + 1;
        if (lane == last) {
          key[q] = next[q];
          r[q] += 1;
        }
      }
    }
    n += 1;
    extra += 1;
    s2 -= drop;
    if (extra % SC_REFRESH == 0) s2 = sum_w2_over_r();
    const double lhs = static_cast<double>(n) * s2;
    more = cv_threshold < 0.0 || lhs > surely_over;
    if (!more && !(lhs < surely_under)) more = cv_exact() > cv_threshold;
    more = more && extra < max_extra;
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

// Exclusive prefix sum over the block's 256 threads; *total = the sum.  part: LDS, four entries (a
// caller that uses it twice passes two arrays).
__device__ __forceinline__ long long block_prefix(long long v, long long* part, long long* total) {
  const int lane = lane_id(), wave = threadIdx.x / MOE_WAVE;
  long long incl = v;
#pragma unroll
  for (int off = 1; off < MOE_WAVE; off <<= 1) {
    const long long up = __shfl_up(incl, off);
    if (lane >= off) incl += up;
  }
  if (lane == MOE_WAVE - 1) part[wave] = incl;
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
  const auto kernel = E <= 64 ? moe::scale_kernel<1> : E <= 128 ? moe::scale_kernel<2> : moe::scale_kernel<4>;
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
// GPU with the smallest aggregated load.  GPU loads are fp64 sums in placement order, and every step
// needs the loads that the step before left: ONE wave runs the steps, lane g holding GPU g's load,
// count and slots, "shortest queue" an arg-min over the lanes with a free slot (upper words of the
// non-negative doubles by DPP, a ballot, lower words only on a tie).  Everything a step needs that does
// not depend on the loads is prepared by the whole block, PL_CHUNK steps at a time, in LDS: the
// order of the experts (all replicas of an expert carry W_e / R_e, so they are placed one after the
// other; ranks by counting, quotients compared exactly as in scale_kernel), and per step the load,
// the warm GPU and the place of the result.  A step is then one LDS read, requested a step ahead,
// and the arg-min.  Measured: 128 replicas of 64 experts on 8 GPUs 110 us with a 64-lane shuffle
// arg-max per expert, one arg-min over 64 lanes of doubles and (warm rounds) one trip to memory per
// step, now 19 us.
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
  __shared__ double key[MOE_MAX_E];
  __shared__ int seg_start[MOE_MAX_E], prev_n[MOE_MAX_E], rep[MOE_MAX_E];
  __shared__ long long prev_start[MOE_MAX_E];    // (the previous round's counts are the caller's: their sum may pass 2^31)
  __shared__ int order[MOE_MAX_E], order_start[MOE_MAX_E + 1];
  __shared__ long long part[3][4];
  const int tid = threadIdx.x, lane = lane_id();
  // thread e: expert e
  const int my_r = tid < E ? min(max(replicas[tid], 1), MOE_MAX_EXTRA_REPLICAS + 1) : 0;
  const int my_p = tid < E && prev_replicas ? max(prev_replicas[tid], 0) : 0;
  const double my_key = tid < E ? static_cast<double>(max(loads[tid], 0)) / static_cast<double>(my_r) : -1.0;
  long long total, dummy;
  seg_start[tid] = static_cast<int>(block_prefix(my_r, part[0], &total));    // (at most 256 * 65537)
  prev_start[tid] = block_prefix(my_p, part[1], &dummy);
  prev_n[tid] = my_p;
  rep[tid] = my_r;
  key[tid] = my_key;
  __syncthreads();
  if (tid < E) {
    int rank = 0;                              // experts before this one: more loaded, or equal and lower
#pragma unroll 8
    for (int e = 0; e < E; ++e) rank += (key[e] > my_key || (key[e] == my_key && e < tid)) ? 1 : 0;
    order[rank] = tid;
  }
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
  for (int first = 0; first < steps; first += PL_CHUNK) {
    const int n = min(PL_CHUNK, steps - first);
    for (int i = tid; i < n; i += 256) {
      const int s = first + i;
      int lo = 0, hi = E - 1;                  // last rank whose first step is <= s
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (order_start[mid] <= s) lo = mid; else hi = mid - 1;
      }
      const int e = order[lo], q = s - order_start[lo];
      int g = -1;
      if (q < prev_n[e]) g = prev_gpu[prev_start[e] + q];
      step[i].w = key[e];
      step[i].warm = g >= 0 && g < G ? g : -1;
      step[i].out = seg_start[e] + q;
    }
    __syncthreads();
    if (tid < MOE_WAVE) {
      unsigned long long room = __ballot(gcount < gslots);
      PlaceStep cur = step[0];
      for (int i = 0; i < n; ++i) {
        const PlaceStep ahead = step[i + 1];   // (past the chunk's last step: read, not used)
        const int wg = __builtin_amdgcn_readfirstlane(cur.warm);
        int g = -1;
        if (wg >= 0 && ((room >> wg) & 1ull)) {
          g = wg;
          ++warm;
        } else {
          const bool free_slot = (room >> lane) & 1ull;
          const uint32_t h = free_slot ? hi32(gload) : 0xFFFFFFFFu;
          const uint32_t least = wave_extreme<false, WIDE>(h);
          if (least != 0xFFFFFFFFu) {
            unsigned long long who = __ballot(h == least);
            if (__popcll(who) > 1) {
              const uint32_t l = h == least ? lo32(gload) : 0xFFFFFFFFu;
              const uint32_t least_lo = wave_extreme<false, WIDE>(l);
              who = __ballot(h == least && l == least_lo);
            }
            g = __ffsll(static_cast<long long>(who)) - 1;
          }
        }
        if (lane == g) {
          gload += cur.w;
          gcount += 1;
        }
        room = __ballot(gcount < gslots);
        if (lane == 0) step[i].warm = g;       // the step's result, in place of its input
        cur = ahead;
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
