// moe_count_and_permute: per-expert token counts (the paper's expert load W_l,
// Sections 3.3 / 4.1), their prefix sum, the stable expert-contiguous permutation
// of the T*k assignments and the row gather that realises the single-GPU "scatter"
// of Section 2.2.
//
// Three launches on the caller's stream (batches of up to DR_MAX_A assignments: rank_direct_kernel
// replaces all three), no host synchronisation:
//   1. hist_kernel   NTH tokens per block; LDS histogram of the block's
//                    assignments -> partial[block][expert]              (integer)
//   2. rank_kernel   same token partition.  Every block sums `partial` to get
//                    counts, offsets and its own base row per expert, then ranks
//                    its assignments with a per-(expert, thread) LDS counter table
//                    and a prefix scan over threads, so the rank of an assignment
//                    is the number of earlier assignments of the same expert: a
//                    stable order, independent of scheduling, no atomics on the
//                    result.
//   3. gather_kernel one wave per token: reads the token row once (16 B per
//                    lane, coalesced), writes it to its k destination rows.
//                    HBM-bound: T*d*b bytes read, T*k*d*b written.
#include <mutex>

#include "moe_internal.h"

namespace moe {

template <int NTH>
__global__ __launch_bounds__(NTH) void hist_kernel(const int32_t* __restrict__ topk_idx, int T,
                                                   int k, int E,
                                                   int32_t* __restrict__ partial) {
  __shared__ int32_t hist[MOE_MAX_E];
  const int tid = threadIdx.x;
  for (int e = tid; e < E; e += NTH) hist[e] = 0;
  __syncthreads();
  // (lanes take neighbouring assignments, whose order does not matter here, eight loads in flight each)
  const int t0 = blockIdx.x * NTH;
  const int64_t n = static_cast<int64_t>(min(NTH, T - t0)) * k;
  const int32_t* first = topk_idx + static_cast<int64_t>(t0) * k;
  constexpr int UNR = 8;
  for (int64_t i0 = tid; i0 < n; i0 += UNR * NTH) {
    int e[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) e[u] = first[min(i0 + u * NTH, n - 1)];
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (i0 + u * NTH < n && static_cast<unsigned>(e[u]) < static_cast<unsigned>(E)) atomicAdd(&hist[e[u]], 1);
  }
  __syncthreads();
  for (int e = tid; e < E; e += NTH) partial[static_cast<int64_t>(blockIdx.x) * E + e] = hist[e];
}

constexpr int RANK_IDS = 8;          // a thread's experts kept in registers (further ones are read twice)

// Dynamic LDS layout: uint16 cnt[E][NTH] | int32 tot[E] | int32 base[E]
template <int NTH>
__global__ __launch_bounds__(NTH) void rank_kernel(const int32_t* __restrict__ topk_idx, int T,
                                                   int k, int E,
                                                   const int32_t* __restrict__ partial, int NB,
                                                   int32_t* __restrict__ counts,
                                                   int32_t* __restrict__ offsets,
                                                   int32_t* __restrict__ dst_row,
                                                   int32_t* __restrict__ src_assign) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint16_t* cnt = reinterpret_cast<uint16_t*>(smem);
  int32_t* tot = reinterpret_cast<int32_t*>(smem + static_cast<size_t>(E) * NTH * 2);
  int32_t* base = tot + E;
  constexpr int NW = NTH / MOE_WAVE;
  constexpr int PER = NTH / MOE_WAVE;  // table entries of one row held by one lane
  const int tid = threadIdx.x;
  const int lane = tid & (MOE_WAVE - 1);
  const int wave = tid / MOE_WAVE;
  const int b = blockIdx.x;
  // Everything the block needs first is requested before the table is cleared: a thread's first RANK_IDS experts and
  // its first share of `partial` (one load after the other, after the clearing, both were trips to memory
  // that nothing covered; 8192 tokens, 64 experts, k = 6: 7.2 -> 6.1 us, with the histogram's neighbouring loads the
  // predictor pass 51.3 -> 49.8; 65536 tokens, k = 2: 5.0, as before)
  const int t = b * NTH + tid;
  const int32_t* row = topk_idx + static_cast<int64_t>(min(t, T - 1)) * k;
  int id[RANK_IDS];
#pragma unroll
  for (int j = 0; j < RANK_IDS; ++j) id[j] = row[min(j, k - 1)];
  auto each_id = [&](auto f) {
    if (t >= T) return;
#pragma unroll
    for (int j = 0; j < RANK_IDS; ++j)
      if (j < k) f(j, id[j]);
    for (int j = RANK_IDS; j < k; ++j) f(j, row[j]);
  };
  const int n = NB * E;
  constexpr int UNR = 8;
  int v[UNR];
  auto load_partial = [&](int i0) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) v[u] = partial[min(i0 + u * NTH, n - 1)];
  };
  load_partial(tid);

  // zero the counter table (16 B per store)
  {
    uint4* z = reinterpret_cast<uint4*>(cnt);
    const int n16 = E * NTH * 2 / 16;
    for (int i = tid; i < n16; i += NTH) z[i] = make_uint4(0, 0, 0, 0);
  }
  // totals per expert and the part that belongs to earlier blocks: every thread takes a strided
  // share of partial[NB][E] (coalesced, several loads in flight) and adds it into LDS; integer
  // sums, so the order of the atomics does not matter
  for (int e = tid; e < E; e += NTH) {
    tot[e] = 0;
    base[e] = 0;
  }
  __syncthreads();
  {
    const int e_step = NTH % E, b_step = NTH / E;
    int e = tid % E, bb = tid / E;               // of entry i0 + u * NTH
    for (int i0 = tid; i0 < n;) {
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        if (i0 + u * NTH < n && v[u] != 0) {
          atomicAdd(&tot[e], v[u]);
          if (bb < b) atomicAdd(&base[e], v[u]);
        }
        e += e_step;
        bb += b_step;
        if (e >= E) {
          e -= E;
          ++bb;
        }
      }
      i0 += UNR * NTH;
      if (i0 < n) load_partial(i0);
    }
  }
  __syncthreads();
  // exclusive scan of tot over experts by wave 0 (E <= 256: at most 4 per lane)
  if (wave == 0) {
    const int per = (E + MOE_WAVE - 1) / MOE_WAVE;
    const int e0 = lane * per;
    int local = 0;
    for (int i = 0; i < per; ++i)
      if (e0 + i < E) local += tot[e0 + i];
    const int incl = wave_scan_add(local);
    int run = incl - local;
    for (int i = 0; i < per; ++i) {
      const int e = e0 + i;
      if (e < E) {
        const int c = tot[e];
        if (b == 0) {
          counts[e] = c;
          offsets[e] = run;
        }
        base[e] += run;
        run += c;
      }
    }
    if (b == 0 && lane == MOE_WAVE - 1) offsets[E] = incl;
  }
  // count this thread's assignments in its private column of the table
  each_id([&](int, int e) {
    if (static_cast<unsigned>(e) < static_cast<unsigned>(E)) cnt[e * NTH + tid] += 1;
  });
  __syncthreads();
  // per expert: exclusive prefix over threads (in place); rows are dealt to waves.  Scans by DPP (by lane
  // shuffles, six trips through the LDS per row: 49152 assignments of 64 experts 10.2 us, so 8.0)
  for (int e = wave; e < E; e += NW) {
    uint16_t* r = cnt + e * NTH + lane * PER;
    uint16_t v[PER];
    int local = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      v[i] = r[i];
      local += v[i];
    }
    const int incl = wave_scan_add(local);
    int run = incl - local;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      r[i] = static_cast<uint16_t>(run);
      run += v[i];
    }
  }
  __syncthreads();
  each_id([&](int j, int e) {
    const int a = t * k + j;
    if (static_cast<unsigned>(e) < static_cast<unsigned>(E)) {
      const int r = cnt[e * NTH + tid];
      cnt[e * NTH + tid] = static_cast<uint16_t>(r + 1);
      const int dst = base[e] + r;
      dst_row[a] = dst;
      src_assign[dst] = a;
    } else {
      dst_row[a] = 0;  // invalid expert index: value unspecified, stays in bounds
    }
  });
}

// Batches of up to DR_MAX_A assignments: one launch does the whole dispatch.  The place of assignment a
// with expert e is the number of assignments b with (expert, b) < (e, a) in lexicographic order, so with
// keys expert << 13 | b it is a plain count of smaller keys, and offsets[e] is the same count for the key
// e << 13: no histogram, no table, no second launch.  Every block keeps all keys in LDS; a wave
// answers two queries in one walk over them (two vector instructions per query and 64 keys), waves
// past the assignments those of expert e and e + 1.  With x_perm a wave also copies the rows of its two
// assignments (COPY).  The count is quadratic: bound by latency up to about 4000 assignments, by the
// vector pipe above.  (Measured, assignments: hist + rank_kernel -> this, us: 1000 (8 experts)
// 9.5 -> 4.8, 4503 (12) 10.1 -> 6.4, 6000 (64) 14.6 -> 7.4, 8192 (8) 9.5 -> 10.0, which sets
// DR_MAX_A; against the one-block kernel that batches of up to 256 took, 256 of 128 experts
// 9.0 -> 4.9; with the row copy, hist + rank + gather_kernel -> this: 2000 assignments, 4 KiB rows, 29.7 ->
// 11.5, 4503, 2 KiB rows, 30.1 -> 16.7, 6000, 8 KiB rows, 46.5 -> 35.6; two or four 16-byte loads per
// lane and row in flight instead of one: up to 4 us slower.  Four queries per wave: up to 0.8 us slower.)
constexpr int DR_THREADS = 512;
constexpr int DR_KEY_BITS = 13;
constexpr int DR_MAX_A = 6144;
static_assert(DR_MAX_A <= 1 << DR_KEY_BITS, "an assignment's number fits its key");
constexpr int DR_STEP = 4 * MOE_WAVE;             // keys a wave compares per LDS read
constexpr uint32_t DR_NO_KEY = 0xFFFFFFFFu;       // not counted by any query

template <bool COPY>
__global__ __launch_bounds__(DR_THREADS) void rank_direct_kernel(
    const int32_t* __restrict__ topk_idx, int A, int E, int k, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ dst_row, int32_t* __restrict__ src_assign,
    const uint4* __restrict__ x, uint4* __restrict__ x_perm, int row16) {
  extern __shared__ __align__(16) uint32_t keys[];        // A rounded up to a multiple of DR_STEP
  const int lane = threadIdx.x & (MOE_WAVE - 1);
  const int steps = (A + DR_STEP - 1) / DR_STEP;
  constexpr int UNR = 8;                                  // loads in flight per thread
  for (int b0 = threadIdx.x; b0 < steps * DR_STEP; b0 += UNR * DR_THREADS) {
    int e[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int b = b0 + u * DR_THREADS;
      e[u] = b < A ? topk_idx[b] : -1;
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int b = b0 + u * DR_THREADS;
      if (b < steps * DR_STEP)
        keys[b] = static_cast<unsigned>(e[u]) < static_cast<unsigned>(E)
                      ? static_cast<uint32_t>(e[u]) << DR_KEY_BITS | static_cast<uint32_t>(b) : DR_NO_KEY;
    }
  }
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * (DR_THREADS / MOE_WAVE) + threadIdx.x / MOE_WAVE);
  constexpr int Q = 2;                                    // queries per wave
  const int a_waves = (A + Q - 1) / Q;
  const bool experts = w >= a_waves;                      // wave-uniform
  const int q0 = experts ? w - a_waves : w * Q;
  if (experts && q0 >= E) return;
  uint32_t key[Q];
  int cnt[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (experts) key[q] = static_cast<uint32_t>(min(q0 + q, E)) << DR_KEY_BITS;
    else key[q] = q0 + q < A ? __builtin_amdgcn_readfirstlane(keys[min(q0 + q, A - 1)]) : DR_NO_KEY;
    cnt[q] = 0;
  }
  for (int s = 0; s < steps; ++s) {
    const uint4 v = *reinterpret_cast<const uint4*>(keys + s * DR_STEP + lane * 4);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      cnt[q] += (v.x < key[q]) + (v.y < key[q]) + (v.z < key[q]) + (v.w < key[q]);
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) cnt[q] = __builtin_amdgcn_readlane(wave_scan_add(cnt[q]), MOE_WAVE - 1);
  if (experts) {
    if (lane == 0) {
      counts[q0] = cnt[1] - cnt[0];
      offsets[q0] = cnt[0];
      if (q0 == E - 1) offsets[E] = cnt[1];
    }
    return;
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int a = q0 + q;
    if (a >= A) break;
    const bool valid = key[q] != DR_NO_KEY;
    // invalid expert index: dst_row's value is unspecified, stays in bounds
    if (lane == 0) dst_row[a] = valid ? cnt[q] : 0;
    if (lane == 0 && valid) src_assign[cnt[q]] = a;
  }
  if (COPY) {
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (q0 + q >= A || key[q] == DR_NO_KEY) cnt[q] = -1;
    for (int c = lane; c < row16; c += MOE_WAVE) {
      uint4 v[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (cnt[q] >= 0) v[q] = x[static_cast<int64_t>((q0 + q) / k) * row16 + c];
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (cnt[q] >= 0) x_perm[static_cast<int64_t>(cnt[q]) * row16 + c] = v[q];
    }
  }
}

// One wave per token.  row16 = row size in 16-byte units.  Where the accesses take the non-temporal hint
// (all measurements in us):
//   OUT_STREAM, the stores: rows written with the default policy stay dirty in the 256 MB memory-side cache.
//     While x and x_perm fit it, and the experts are compute-bound, that is where the up-projection finds
//     them (whole four-call layer, with the hint / without: 64-expert shape at 3500 / 6000 tokens
//     509 / 478 and 658 / 635, skewed at 8192 tokens 948 / 939, llama4 shape at 8192 tokens 1794 / 1765).  Past
//     that size the next large read pays for writing them back (route + permute + combine: 65536
//     tokens, d = 4096, k = 2 632 / 698; 24000 tokens, d = 5120, k = 1 216 / 251), and where an FFN of few
//     rows per expert streams its weights, the write-backs cost that stream (128-expert shape at 1500 / 4096
//     tokens, 94 and 256 rows per expert, 987 / 1049 and 1453 / 1488).
//   X_STREAM, the loads: where x fits the cache, the routing has just left it there (the same three calls,
//     with / without: x of 245 MB, 24000 tokens, d = 5120, k = 1 234 / 216; 295 MB, 36000 tokens, d = 4096,
//     k = 2 337 / 347; 537 MB 634 / 675), unless x_perm's rows push it out meanwhile (d = 4096: 20000
//     tokens, k = 4, 819 MB with x_perm, 312 / 312; 32000, k = 4, 1311 MB 488 / 502; 15000, k = 8, 1106 MB 485 / 494).
constexpr int64_t MEMORY_SIDE_CACHE_BYTES = int64_t(256) << 20;
constexpr int WEIGHT_BOUND_ROWS = 256;     // mean rows per expert up to which the FFN waits for its weights
template <bool X_STREAM, bool OUT_STREAM>
__global__ __launch_bounds__(256) void gather_kernel(const uint4* __restrict__ x,
                                                     const int32_t* __restrict__ dst_row,
                                                     uint4* __restrict__ x_perm, int T, int k,
                                                     int row16, int A) {
  const int lane = threadIdx.x & (MOE_WAVE - 1);
  const int t = blockIdx.x * (256 / MOE_WAVE) + threadIdx.x / MOE_WAVE;
  if (t >= T) return;
  int my_dst = 0;
  if (lane < k) my_dst = dst_row[static_cast<int64_t>(t) * k + lane];
  if (static_cast<unsigned>(my_dst) >= static_cast<unsigned>(A)) my_dst = 0;
  const uint4* src = x + static_cast<int64_t>(t) * row16;
  constexpr int UNR = 4;   // 16-byte loads in flight per lane (two: as fast or up to 17 % slower)
  for (int c0 = 0; c0 < row16; c0 += UNR * MOE_WAVE) {
    uint4 v[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int c = c0 + u * MOE_WAVE + lane;
      if (c < row16) v[u] = X_STREAM ? nt_load(src + c) : src[c];
    }
    for (int j = 0; j < k; ++j) {
      const int dst = __shfl(my_dst, j);
      uint4* out = x_perm + static_cast<int64_t>(dst) * row16;
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int c = c0 + u * MOE_WAVE + lane;
        if (c >= row16) continue;
        if (OUT_STREAM) nt_store(out + c, v[u]);
        else out[c] = v[u];
      }
    }
  }
}

static int dispatch_threads(int E) { return E <= 128 ? 256 : 128; }

}  // namespace moe

extern "C" int moe_workspace_bytes(const moe_shape_t* shape, size_t* out_bytes) {
  const int rc = moe::check_shape(shape);
  if (rc != MOE_OK) return rc;
  if (!out_bytes) return MOE_ERR_INVALID_ARG;
  const int nth = moe::dispatch_threads(shape->E);
  const int64_t nb = (static_cast<int64_t>(shape->T) + nth - 1) / nth;
  size_t bytes = static_cast<size_t>(nb > 0 ? nb : 1) * shape->E * sizeof(int32_t);
  // moe_route_ws keeps T x E fp32 scores and T + E norms between its two kernels for small batches
  if (shape->T <= MOE_ROUTE_WS_MAX_T) {
    const size_t route_bytes =
        (static_cast<size_t>(shape->T) * shape->E + shape->T + shape->E) * sizeof(float);
    if (route_bytes > bytes) bytes = route_bytes;
  }
  *out_bytes = (bytes + 255) & ~static_cast<size_t>(255);
  return MOE_OK;
}

namespace moe {

// Bytes of partial[blocks][E] that the two-launch dispatch keeps between hist_kernel and rank_kernel.
static size_t dispatch_partial_bytes(const moe_shape_t* shape) {
  const int nth = dispatch_threads(shape->E);
  const int64_t nb = (static_cast<int64_t>(shape->T) + nth - 1) / nth;
  return static_cast<size_t>(nb > 0 ? nb : 1) * shape->E * sizeof(int32_t);
}

// Everything after the checks of the workspace: `partial` holds dispatch_partial_bytes() bytes.
// hist_kernel writes every entry of it that rank_kernel reads, so its old contents do not matter.
static int count_and_permute_impl(const moe_shape_t* shape, const void* x, const int32_t* topk_idx,
                                  int32_t* counts, int32_t* offsets, int32_t* dst_row,
                                  int32_t* src_assign, void* x_perm, int32_t* partial,
                                  hipStream_t st) {
  const int T = shape->T, k = shape->k, E = shape->E;
  const int nth = dispatch_threads(E);
  const int grid = (T + nth - 1) / nth;
  const size_t lds = static_cast<size_t>(E) * nth * 2 + static_cast<size_t>(E) * 8;
  const int64_t A = static_cast<int64_t>(T) * k;
  bool copy = T > 0 && x_perm;
  const int row16 = static_cast<int>(static_cast<int64_t>(shape->d) * elem_bytes(shape->dtype) / 16);
  if (A <= DR_MAX_A) {                            // (also A = 0: counts and offsets become zeros)
    const int lds_keys = static_cast<int>((A + DR_STEP - 1) / DR_STEP) * DR_STEP * 4;
    const int blocks = static_cast<int>(((A + 1) / 2 + E + DR_THREADS / MOE_WAVE - 1) / (DR_THREADS / MOE_WAVE));
    hipLaunchKernelGGL(copy ? rank_direct_kernel<true> : rank_direct_kernel<false>, dim3(blocks), dim3(DR_THREADS),
                       lds_keys, st, topk_idx, static_cast<int>(A), E, k, counts, offsets, dst_row, src_assign,
                       static_cast<const uint4*>(x), static_cast<uint4*>(x_perm), row16);
    copy = false;
  } else if (nth == 256) {
    static LdsOnce once;
    if (ensure_dynamic_lds(once, reinterpret_cast<const void*>(rank_kernel<256>),
                           128 * 256 * 2 + 128 * 8) != MOE_OK)
      return MOE_ERR_HIP;
    hipLaunchKernelGGL(hist_kernel<256>, dim3(grid), dim3(256), 0, st, topk_idx, T, k, E, partial);
    hipLaunchKernelGGL(rank_kernel<256>, dim3(grid), dim3(256), lds, st, topk_idx, T, k, E, partial,
                       grid, counts, offsets, dst_row, src_assign);
  } else {
    static LdsOnce once;
    if (ensure_dynamic_lds(once, reinterpret_cast<const void*>(rank_kernel<128>),
                           256 * 128 * 2 + 256 * 8) != MOE_OK)
      return MOE_ERR_HIP;
    hipLaunchKernelGGL(hist_kernel<128>, dim3(grid), dim3(128), 0, st, topk_idx, T, k, E, partial);
    hipLaunchKernelGGL(rank_kernel<128>, dim3(grid), dim3(128), lds, st, topk_idx, T, k, E, partial,
                       grid, counts, offsets, dst_row, src_assign);
  }
  if (copy) {
    const int64_t x_bytes = static_cast<int64_t>(T) * row16 * 16;
    const int64_t total_bytes = x_bytes * (k + 1);
    const bool x_stream = x_bytes > MEMORY_SIDE_CACHE_BYTES || total_bytes > 3 * MEMORY_SIDE_CACHE_BYTES;
    const bool out_stream = total_bytes > MEMORY_SIDE_CACHE_BYTES || A / E <= WEIGHT_BOUND_ROWS;
    const auto kernel = x_stream ? gather_kernel<true, true>
                        : out_stream ? gather_kernel<false, true> : gather_kernel<false, false>;
    hipLaunchKernelGGL(kernel, dim3((T + 3) / 4), dim3(256), 0, st,
                       static_cast<const uint4*>(x), dst_row, static_cast<uint4*>(x_perm), T, k,
                       row16, T * k);
  }
  return launch_status();
}

static int check_dispatch_args(const moe_shape_t* shape, const void* x, const int32_t* topk_idx,
                               const int32_t* counts, const int32_t* offsets, const int32_t* dst_row,
                               const int32_t* src_assign, const void* x_perm) {
  const int rc = check_shape(shape);
  if (rc != MOE_OK) return rc;
  if (!counts || !offsets) return MOE_ERR_INVALID_ARG;
  if (shape->T > 0 && (!topk_idx || !dst_row || !src_assign)) return MOE_ERR_INVALID_ARG;
  if (shape->T > 0 && x_perm && (!x || !aligned16(x) || !aligned16(x_perm))) return MOE_ERR_INVALID_ARG;
  return MOE_OK;
}

// ---- the dispatch for callers that cannot allocate ------------------------------------------
// The block histograms of moe_count_and_permute_static live in this array instead of a caller's
// workspace: one copy per GPU, held for the life of the process.  In host code the array's name
// is only a handle for the runtime: the address the kernels are given is looked up once per
// device with hipGetSymbolAddress and kept.
static __device__ __align__(256) unsigned char scratch[MOE_STATIC_SCRATCH_BYTES];
static void* g_scratch_addr[MOE_MAX_DEVICES] = {};
static std::mutex g_scratch_mutex;

static int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MOE_MAX_DEVICES) return MOE_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return MOE_ERR_HIP;
    }
    g_scratch_addr[dev] = p;
  }
  *out = g_scratch_addr[dev];
  return MOE_OK;
}

}  // namespace moe

extern "C" int moe_count_and_permute(const moe_shape_t* shape, const void* x,
                                     const int32_t* topk_idx, int32_t* counts, int32_t* offsets,
                                     int32_t* dst_row, int32_t* src_assign, void* x_perm,
                                     void* workspace, size_t workspace_bytes, void* hip_stream) {
  const int rc = moe::check_dispatch_args(shape, x, topk_idx, counts, offsets, dst_row, src_assign, x_perm);
  if (rc != MOE_OK) return rc;
  size_t need = 0;
  moe_workspace_bytes(shape, &need);
  if (!workspace || !moe::aligned16(workspace)) return MOE_ERR_INVALID_ARG;
  if (workspace_bytes < need) return MOE_ERR_WORKSPACE;
  return moe::count_and_permute_impl(shape, x, topk_idx, counts, offsets, dst_row, src_assign, x_perm,
                                     static_cast<int32_t*>(workspace),
                                     static_cast<hipStream_t>(hip_stream));
}

extern "C" int moe_count_and_permute_static(const moe_shape_t* shape, const void* x,
                                            const int32_t* topk_idx, int32_t* counts,
                                            int32_t* offsets, int32_t* dst_row, int32_t* src_assign,
                                            void* x_perm, void* hip_stream) {
  const int rc = moe::check_dispatch_args(shape, x, topk_idx, counts, offsets, dst_row, src_assign, x_perm);
  if (rc != MOE_OK) return rc;
  // the batch must fit the fixed array: ceil(T / 256) * E * 4 bytes (blocks of 128 tokens above 128 experts)
  if (moe::dispatch_partial_bytes(shape) > MOE_STATIC_SCRATCH_BYTES) return MOE_ERR_WORKSPACE;
  void* partial = nullptr;
  if (moe::static_scratch(&partial) != MOE_OK) return MOE_ERR_HIP;
  return moe::count_and_permute_impl(shape, x, topk_idx, counts, offsets, dst_row, src_assign, x_perm,
                                     static_cast<int32_t*>(partial),
                                     static_cast<hipStream_t>(hip_stream));
}
