// moe_combine: y[t,:] = sum_{j<k} topk_w[t,j] * y_perm[dst_row[t*k+j], :]
// The single-GPU form of the "gather" of Section 2.2 (collect the expert outputs
// and put them back in token order), fused with the routing-weight scaling of
// y = sum_k g_k(x) E_k(x).  Written as a gather per output token rather than a
// scatter-add: every output element is produced by exactly one lane, summed in
// fp32 in ascending j, so the result is deterministic and needs no atomics and no
// zero-fill of y.  HBM-bound: reads T*k*d*b, writes T*d*b.
#include "moe_internal.h"

namespace moe {
// Streaming accesses: y_perm is read once and y written once by this call, so neither should
// displace anything in the caches (measured on 65536 tokens, d = 4096, k = 2: 312 -> 280 us; the
// 64-expert layer at 8192 tokens 43 -> 39.5 us; the small batches unchanged).
//
// One wave per (token, slab of 64*UNR 16-byte column chunks).  The blocks of a token's slabs are
// neighbours, so a row's pieces travel together; in a two-dimensional grid the second slab of every token
// came after the first slab of all of them.  (Measured, neighbours and UNR = 2 against that
// grid and UNR = 4: 65536 tokens, d = 4096, k = 2 270 -> 251 us, 6.4 TB/s; 30000 tokens, d = 5120, k = 1
// 111 -> 99 us; 32 to 8192 tokens within 0.4 us.  UNR = 8: 265 / 128 us.)  Blocks are dealt to the
// eight XCDs in turn, so with an even number of slabs some XCDs would get the full slabs and others the
// short last ones: combine_unr avoids that.
template <bool BF16, int UNR>
__global__ __launch_bounds__(256) void combine_kernel(const uint4* __restrict__ y_perm,
                                                      const int32_t* __restrict__ dst_row,
                                                      const float* __restrict__ topk_w,
                                                      uint4* __restrict__ y, int T, int k,
                                                      int row16, int A, int slabs, int t0) {
  const int lane = threadIdx.x & (MOE_WAVE - 1);
  const int t = t0 + blockIdx.x / slabs * (256 / MOE_WAVE) + threadIdx.x / MOE_WAVE;
  if (t >= T) return;
  int my_dst = 0;
  float my_w = 0.f;
  if (lane < k) {
    my_dst = dst_row[static_cast<int64_t>(t) * k + lane];
    my_w = topk_w[static_cast<int64_t>(t) * k + lane];
  }
  if (static_cast<unsigned>(my_dst) >= static_cast<unsigned>(A)) my_dst = 0;
  constexpr int NACC = BF16 ? 8 : 4;
  const int c_begin = blockIdx.x % slabs * (UNR * MOE_WAVE);
  float acc[UNR][NACC];
#pragma unroll
  for (int u = 0; u < UNR; ++u)
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[u][i] = 0.f;
  // The rows of JB experts are requested before the first is used (their addresses only depend
  // on the map, and a wave that waits for one row at a time is latency-bound when there are few
  // tokens); the sum still runs in ascending j.
  constexpr int JB = 4;
  for (int j0 = 0; j0 < k; j0 += JB) {
    uint4 v[JB][UNR];
    float w[JB];
#pragma unroll
    for (int jj = 0; jj < JB; ++jj) {
      const int j = min(j0 + jj, k - 1);
      const int src = __shfl(my_dst, j);
      w[jj] = __shfl(my_w, j);
      const uint4* in = y_perm + static_cast<int64_t>(src) * row16;
      if (j0 + jj < k) {                            // wave-uniform
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const int c = c_begin + u * MOE_WAVE + lane;
          v[jj][u] = nt_load(in + min(c, row16 - 1));
        }
      }
    }
#pragma unroll
    for (int jj = 0; jj < JB; ++jj) {
      if (j0 + jj < k) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const uint4 q = v[jj][u];
          const float ww = w[jj];
          if (BF16) {
            acc[u][0] = fmaf(ww, bf16lo(q.x), acc[u][0]);
            acc[u][1] = fmaf(ww, bf16hi(q.x), acc[u][1]);
            acc[u][2] = fmaf(ww, bf16lo(q.y), acc[u][2]);
            acc[u][3] = fmaf(ww, bf16hi(q.y), acc[u][3]);
            acc[u][4] = fmaf(ww, bf16lo(q.z), acc[u][4]);
            acc[u][5] = fmaf(ww, bf16hi(q.z), acc[u][5]);
            acc[u][6] = fmaf(ww, bf16lo(q.w), acc[u][6]);
            acc[u][7] = fmaf(ww, bf16hi(q.w), acc[u][7]);
          } else {
            acc[u][0] = fmaf(ww, __uint_as_float(q.x), acc[u][0]);
            acc[u][1] = fmaf(ww, __uint_as_float(q.y), acc[u][1]);
            acc[u][2] = fmaf(ww, __uint_as_float(q.z), acc[u][2]);
            acc[u][3] = fmaf(ww, __uint_as_float(q.w), acc[u][3]);
          }
        }
      }
    }
  }
  uint4* out = y + static_cast<int64_t>(t) * row16;
#pragma unroll
  for (int u = 0; u < UNR; ++u) {
    const int c = c_begin + u * MOE_WAVE + lane;
    if (c < row16) {
      uint4 v;
      if (BF16) {
        v.x = pack_bf16x2(acc[u][0], acc[u][1]);
        v.y = pack_bf16x2(acc[u][2], acc[u][3]);
        v.z = pack_bf16x2(acc[u][4], acc[u][5]);
        v.w = pack_bf16x2(acc[u][6], acc[u][7]);
      } else {
        v.x = __float_as_uint(acc[u][0]);
        v.y = __float_as_uint(acc[u][1]);
        v.z = __float_as_uint(acc[u][2]);
        v.w = __float_as_uint(acc[u][3]);
      }
      nt_store(out + c, v);
    }
  }
}

// UNR for rows of row16 chunks: the least of 2, 3, 4 that cuts them into an odd number of slabs, else 2.
// (Measured, 15000 tokens, k = 2, UNR = 2 / 3 / 4 in us: 136 chunks 21.3 / 17.2 / 17.7; 193: 27.7 / 32.6 / 24.0;
// 257: 33.8 / 36.9 / 41.9; 385: 50.6 / 48.5 / 51.8; 577: 70.8 / 73.4 / 69.5; 641: 86.1 / 80.0 / 75.9;
// 900: 107.6 / 102.2 / 108.4; 1025: 123.7 / 129.4 / 120.8.  Where the slabs are all full, 256, 384, 512 and
// 768 chunks, every choice is within 1 % of the others but 3 at 256.)
static int combine_unr(int row16) {
  for (int unr = 2; unr <= 4; ++unr)
    if ((row16 + unr * MOE_WAVE - 1) / (unr * MOE_WAVE) % 2 == 1) return unr;
  return 2;
}

template <bool BF16>
static int launch_combine(const moe_shape_t* shape, const void* y_perm, const int32_t* dst_row, const float* topk_w,
                          void* y, hipStream_t st) {
  const int T = shape->T;
  const int row16 = static_cast<int>(static_cast<int64_t>(shape->d) * elem_bytes(shape->dtype) / 16);
  const int unr = combine_unr(row16);
  const int slabs = (row16 + unr * MOE_WAVE - 1) / (unr * MOE_WAVE);
  const auto kernel = unr == 2 ? combine_kernel<BF16, 2> : unr == 3 ? combine_kernel<BF16, 3> : combine_kernel<BF16, 4>;
  // one launch, unless the grid would pass the 2^32 threads that a launch may have
  const int64_t per_launch = static_cast<int64_t>(((1 << 24) - 1) / slabs) * 4;
  for (int64_t t0 = 0; t0 < T; t0 += per_launch) {
    const int64_t n = T - t0 < per_launch ? T - t0 : per_launch;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((n + 3) / 4 * slabs)), dim3(256), 0, st,
                       static_cast<const uint4*>(y_perm), dst_row, topk_w, static_cast<uint4*>(y), T,
                       shape->k, row16, T * shape->k, slabs, static_cast<int>(t0));
  }
  return launch_status();
}

}  // namespace moe

extern "C" int moe_combine(const moe_shape_t* shape, const void* y_perm, const int32_t* dst_row,
                           const float* topk_w, void* y, void* hip_stream) {
  const int rc = moe::check_shape(shape);
  if (rc != MOE_OK) return rc;
  if (shape->T == 0) return MOE_OK;
  if (!y_perm || !dst_row || !topk_w || !y) return MOE_ERR_INVALID_ARG;
  if (!moe::aligned16(y_perm) || !moe::aligned16(y)) return MOE_ERR_INVALID_ARG;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  return shape->dtype == MOE_BF16 ? moe::launch_combine<true>(shape, y_perm, dst_row, topk_w, y, st)
                                  : moe::launch_combine<false>(shape, y_perm, dst_row, topk_w, y, st);
}
