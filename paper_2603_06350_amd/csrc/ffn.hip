// moe_grouped_ffn: the expert computation that dominates the MoE layer (Section 3.2).
// For every expert e and row r of its segment [offsets[e], offsets[e+1]):
//   h[r] = silu(W1_e x_perm[r]) * (W3_e x_perm[r]),   y_perm[r] = W2_e h[r].
// The activation rows come either from a permuted copy x_perm, or straight from x through the
// dispatch's src_assign map (moe_grouped_ffn_gather: row r is x[src_assign[r] / k]); the map only
// changes the per-lane row offset of the activation loads.
//
// Two GEMMs: a gated one (W1 and W3 tiles side by side, SwiGLU applied to the fp32
// accumulators, h stored once) and a plain one for W2.  Both are ragged grouped
// GEMMs, one launch each: the tile list is derived on the device from `offsets`, so the host
// never learns the expert loads.
//   an expert's c rows are cut into ceil(c / bm) tiles of nearly equal height (multiples of 16 rows;
//   bm is 320, less where experts hold few rows: most_tile_rows), each against 256 weight rows;
//   the height of a tile, or of the expert's highest, then picks its pipeline (decode_tile):
//   up to 64 rows   ring tile (ffn_ring_tile): paced by the weight stream, four-stage LDS ring;
//   65 and more     even tile (ffn_even_tile): hand-ordered MFMA pipeline, two activation buffers and
//                   as many weight buffers as the LDS holds beside them (four, three or two).
//   A tile takes a whole compute unit, so tiles of a last round that is at most half full are cut
//   into pieces for the idle units: low ones along the weight rows, high ones along their own rows.
//
// moe_grouped_ffn_ws brings a workspace of fp32 partial tiles: a tile takes a whole compute unit,
// so a GEMM runs in rounds of the chip, and when the last round of a GEMM with a long reduction
// is at most half full its tiles are computed as 2 to 4 parts of the K range on the idle units
// and added up, in part order, by a second small launch.
//
// bf16 kernels (gfx950): 512 threads = 8 waves, two per SIMD.  K step 64: both
// operands are K-contiguous, so a tile row is 128 B = eight 16-byte chunks.  Tiles go
// global -> LDS with 16-byte-per-lane buffer loads that write LDS directly (no register
// staging); a wave instruction fills 8 rows, and the chunk a lane fetches is
// XOR-swizzled by row so that the 16-byte LDS reads of a 16-row MFMA operand are
// bank-conflict free.  The weight fragment is the MFMA "A" operand and the activation
// fragment "B": a lane then owns 4 consecutive output columns of one output row.
// v_mfma_f32_16x16x32_bf16, fp32 accumulators (on this chip it sustains a higher rate
// than the 32x32x16 form).
//
// Work-group ids are remapped so that each XCD (ids are dealt round-robin to the 8
// XCDs) walks a contiguous range of the tile list with the m-tiles of one weight
// panel adjacent: CUs that share an L2 share weight tiles.
//
// fp32 layers: ffn_f32_kernel, smaller tiles, on the fp32 matrix instruction or on three bf16 pieces per value.
// Layers so wide that the MFMA kernels' 32-bit offsets do not reach over a tile: ffn_wide_kernel.
#include <type_traits>

#include "moe_internal.h"

namespace moe {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

constexpr int BK_ELEMS = 64;    // K elements per stage of the MFMA kernels

struct GemmArgs {
  const void* a;    // activations [rows, K]
  const void* b0;   // gated: W1 [E,N,K]   plain: W2 [E,N,K]
  const void* b1;   // gated: W3 [E,N,K]   plain: unused
  void* out;        // [rows, N]
  const int32_t* offsets;
  int E, K, N;
  int n_tiles;      // tiles along N
  int bn;           // output columns of a whole tile
  int rows;         // T*k; row ranges read from `offsets` are clamped to it
  int bm;           // most rows of a tile
  // Gathered activations: row r of the GEMM is row src_assign[r] / k_div of `a` (the token that
  // assignment r belongs to) instead of row r itself.  nullptr = `a` is already permuted.
  const int32_t* src_assign;
  int k_div;
  int a_rows;       // rows of `a` (gathered row numbers are clamped to it)
  int n_cu;         // compute units of the device (tiles are split by rounds of it)
  // Split tiles (kernels built with SPLIT only): fp32 partial tiles, one slot per compute unit.
  // nullptr: no tile is split.  split_phase 0: the GEMM itself; 1: the launch after it that adds
  // up the parts of every split tile and stores it.
  float* split_ws;
  int split_phase;
  // Scattered, scaled output (plain GEMM of a k = 1 layer: the combine folded into the store):
  // GEMM row r goes to row out_map[r] of `out`, multiplied by out_scale[out_map[r]] before the
  // one rounding.  nullptr = row r of `out`, unscaled.
  const int32_t* out_map;
  const float* out_scale;
  int out_rows;     // rows of `out` (mapped row numbers are clamped to it)
  // Launches without split_ws: tiles of a last round that is at most half full are cut into pieces
  // for the idle units (the grid has a round of extra blocks).
  int tail_split;
  int few_buffers;  // up-projections: experts of several tiles keep two weight buffers (see tile_mi)
};

constexpr int SPLIT_SLOT_FLOATS = 320 * 256;   // one partial tile (the largest: 320 x 256 fp32)
constexpr int SPLIT_MAX_PARTS = 4;
constexpr int SPLIT_MIN_STAGES = 8;            // K stages a part must keep

// Row of `a` that holds GEMM row r.
__device__ __forceinline__ int a_row_of(const GemmArgs& p, int r) {
  if (!p.src_assign) return r;
  const int t = p.src_assign[r] / p.k_div;
  return min(max(t, 0), p.a_rows - 1);
}

struct TileCoord {
  int e, m_begin, m_end;
  int n0;      // first output column
  int n_pieces;  // 2, 4: this is a piece with that share of the whole tile's weight rows
  // K split of a tile of the last, partial round (nparts == 1: the whole K range)
  int part, nparts;
  int pslot;   // partial-tile slot of this part; the parts of a tile have consecutive slots
  int sharers; // tiles and pieces of tiles of this expert that read the same weight rows
  int height;  // rows that pick the pipeline
};
constexpr int TAIL_MAX_PIECES = 4;
// Tiles of at most RING_ROWS rows have little arithmetic per weight byte and are paced by memory
// latency, which the ring pipeline's equal depth for both operands hides best.
constexpr int RING_ROWS = 64;
// Tiles of the last round up to this height are cut along the weight rows: every weight byte is
// still requested once, and these tiles wait for weights.  Higher tiles are cut along their own rows:
// they wait for the matrix pipe, and a piece then takes a pipeline that a whole tile takes too.
constexpr int NSPLIT_ROWS = 128;
constexpr int WGT_NT_MAX_SHARERS = 2;

// Maps a work-group to (expert, row range, n-tile).  Every wave computes this on its
// own from the device-resident offsets; returns false if the group has no tile.
// An expert with c rows has ceil(c / bm) tiles; the segment's 16-row sub-tiles are dealt to them evenly.
// Tile order: expert-major, then n-tile, then m-tile (m fastest), cut into 8 contiguous ranges,
// one per XCD.
// BY_EXPERT: tiles of 129 and more rows take the pipeline that the highest tile of their expert needs,
// otherwise each the one for its own rows.  Tiles that read the same weight rows side by side
// with the non-temporal hint have to keep pace, or the second one finds them gone from the L2; in two
// different pipelines they drift apart.  (Measured at 500 to 530 rows per expert, where most
// experts are a tile below and one above 256 rows, by expert against by own rows: llama4 shape at 8480
// tokens 1925 -> 1830 us, phi shape at 4000 tokens 1115 -> 1095, down-projection of the Mixtral shape at 2000
// tokens 407 -> 389.  Where weight rows stay in the L2, !WNT, the third weight buffer of the lower tiles is
// worth more: 64-expert shape at 8192 tokens, down-projection 266 us by own rows, 273 by expert.  Low tiles
// by expert too: skewed 64-expert layer at 200 to 700 tokens 3 to 4 % slower, Mixtral shape at 480 tokens
// 4 %, at 260 and 360 tokens 1 to 2 % faster.)
template <bool SPLIT = false, bool BY_EXPERT = false>
__device__ __forceinline__ bool decode_tile(const GemmArgs& p, TileCoord& tc) {
  const int32_t* __restrict__ offsets = p.offsets;
  const int E = p.E, n_tiles = p.n_tiles, bm = p.bm;
  const int lane = lane_id();
  const int per = (E + MOE_WAVE - 1) / MOE_WAVE;  // <= 4
  const int e0 = lane * per;
  int mt[4], ob[4], oe[4];                       // tiles, first and end row of this lane's experts
  int local = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = e0 + i;
    ob[i] = 0;
    oe[i] = 0;
    mt[i] = 0;
    if (i < per && e < E) {
      ob[i] = offsets[e];
      oe[i] = offsets[e + 1];
      mt[i] = (max(oe[i] - ob[i], 0) + bm - 1) / bm;
    }
    local += mt[i];
  }
  // prefix sum over the experts (lane order = expert order)
  const int incl = wave_scan_add(local);
  // (tile counts fit 32 bits: the host refuses grids beyond 2^31 - 1 blocks, and a grid is an
  // upper bound of its tile count)
  const int total = __builtin_amdgcn_readlane(incl, MOE_WAVE - 1) * n_tiles;
  const int per_xcd = (total + 7) / 8;
  const int xcd = blockIdx.x & 7;
  const int slot = blockIdx.x >> 3;
  int vid = xcd * per_xcd + slot;
  tc.part = 0;
  tc.nparts = 1;
  tc.pslot = 0;
  int m_pieces = 1, m_piece = 0;
  if (SPLIT && p.split_ws) {
    // The tiles of an XCD's range run in rounds of its compute units.  If the last round is at
    // most half full, its tiles are cut along K into as many parts as fit the idle units (every
    // block of both launches takes the same decision from the same numbers); the grid of the GEMM
    // has a round of extra blocks for the parts.
    const int cus_x = max(1, (p.n_cu > 0 ? p.n_cu : 256) / 8);
    const int full_x = per_xcd / cus_x * cus_x;
    const int tail_x = per_xcd - full_x;
    int parts = 1;
    if (tail_x > 0 && 2 * tail_x <= cus_x)
      parts = min(min(cus_x / tail_x, SPLIT_MAX_PARTS), (p.K / BK_ELEMS) / SPLIT_MIN_STAGES);
    if (parts < 2) parts = 1;
    if (p.split_phase == 1) {
      // the summing launch: block (xcd, t) takes split tile t of the XCD's last round
      if (parts == 1 || slot >= tail_x) return false;
      vid = xcd * per_xcd + full_x + slot;
      tc.nparts = parts;
      tc.pslot = xcd * cus_x + slot * parts;
    } else if (slot >= full_x) {
      const int j = slot - full_x;
      const int t_local = j / parts;
      if (t_local >= tail_x) return false;
      vid = xcd * per_xcd + full_x + t_local;
      tc.part = j - t_local * parts;
      tc.nparts = parts;
      tc.pslot = xcd * cus_x + j;                // j < tail_x * parts <= cus_x
    }
    if (vid >= total) return false;
  } else if (p.tail_split && slot + max(1, (p.n_cu > 0 ? p.n_cu : 256) / 8) >= per_xcd) {
    // No workspace: the tiles of a last round that is at most half full are cut along the weight rows
    // (up to NSPLIT_ROWS high) or along their own rows (each piece then streams the whole weight tile, out
    // of the L2, which its sister pieces fill at the same time).  The outputs are the same bits: an
    // element's sum does not depend on what shares its tile.  (Only blocks of the last two rounds come here: the
    // integer divisions below cost a tile of the rounds before them half a percent of its time.)
    const int cus_x = max(1, (p.n_cu > 0 ? p.n_cu : 256) / 8);
    const int full_x = per_xcd / cus_x * cus_x;
    const int tail_x = per_xcd - full_x;
    if (slot >= full_x) {
      if (tail_x > 0 && 2 * tail_x <= cus_x) m_pieces = min(cus_x / tail_x, TAIL_MAX_PIECES);
      const int j = slot - full_x;
      const int t_local = j / m_pieces;
      if (t_local >= tail_x) return false;
      vid = xcd * per_xcd + full_x + t_local;
      m_piece = j - t_local * m_pieces;
    }
    if (vid >= total) return false;
  } else if (slot >= per_xcd || vid >= total) {
    return false;
  }
  int run = incl - local;
  int found_e = -1, found_local = 0, found_mt = 1, found_ob = 0, found_oe = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int s = run * n_tiles;
    if (mt[i] > 0 && vid >= s && vid < s + mt[i] * n_tiles) {
      found_e = e0 + i;
      found_local = vid - s;
      found_mt = mt[i];
      found_ob = ob[i];
      found_oe = oe[i];
    }
    run += mt[i];
  }
  const unsigned long long who = __ballot(found_e >= 0);
  if (who == 0ull) return false;  // inconsistent offsets: no tile
  const int src = __ffsll(static_cast<long long>(who)) - 1;   // wave-uniform: reads of that lane
  const int e = __builtin_amdgcn_readlane(found_e, src);
  const int loc = __builtin_amdgcn_readlane(found_local, src);
  const int m_tiles = __builtin_amdgcn_readlane(found_mt, src);
  const int m_idx = loc % m_tiles;
  // the lane that owns the expert already holds its row range: no second trip to memory
  const int seg_begin = max(__builtin_amdgcn_readlane(found_ob, src), 0);
  const int seg_end = min(__builtin_amdgcn_readlane(found_oe, src), p.rows);
  tc.e = e;
  tc.n0 = loc / m_tiles * p.bn;
  tc.n_pieces = 1;
  tc.sharers = m_tiles;
  // The segment's 16-row sub-tiles are dealt in pairs: a tile's sub-tiles go to four wave rows,
  // and wave rows 0, 2 and 1, 3 share their SIMDs, so a tile with an odd number of sub-tiles is
  // as slow as one with the next even number.  67 sub-tiles become 17, 16, 16, 18 (9 + 8 + 8 + 9
  // per SIMD pair), not 16, 17, 17, 17 (8 + 9 + 9 + 9).  An odd one out goes to the first tile,
  // which has the fewest pairs (so no tile exceeds 20 sub-tiles).
  const int sub = (seg_end - seg_begin + 15) / 16;
  const int pairs = sub >> 1, odd = sub & 1;
  const int b0 = m_idx == 0 ? 0 : 2 * (m_idx * pairs / m_tiles) + odd;
  const int b1 = 2 * ((m_idx + 1) * pairs / m_tiles) + odd;
  int s0 = b0, s1 = b1;
  int top = b1 - b0;
  if (BY_EXPERT && m_tiles > 1 && top > NSPLIT_ROWS / 16) {     // (the division is skipped where it decides nothing)
    const int q = pairs / m_tiles;
    top = max(2 * (q + (q * m_tiles < pairs ? 1 : 0)), 2 * q + odd);
  }
  if (m_pieces > 1) {
    const int n_sub = b1 - b0;
    if (n_sub <= NSPLIT_ROWS / 16) {
      const int pieces = m_pieces >= 4 && n_sub <= RING_ROWS / 16 ? 4 : 2;
      if (m_piece >= pieces) return false;
      tc.n_pieces = pieces;
      tc.n0 += m_piece * (p.bn / pieces);
      if (tc.n0 >= p.N) return false;
    } else {
      const int pieces = min(m_pieces, max(1, n_sub / 4));    // a piece keeps 64 rows or more
      if (m_piece >= pieces) return false;
      tc.sharers = m_tiles + pieces - 1;
      s0 = b0 + m_piece * n_sub / pieces;
      s1 = b0 + (m_piece + 1) * n_sub / pieces;
      top = s1 - s0;
    }
  }
  tc.m_begin = seg_begin + s0 * 16;
  tc.m_end = min(seg_end, seg_begin + s1 * 16);
  tc.height = BY_EXPERT ? top * 16 : tc.m_end - tc.m_begin;
  return tc.m_begin < tc.m_end;
}

// silu(g) * u.  EXACT: silu first, by expf and a true division (fp32 layers, and bf16 layers whose widths
// are multiples of 8 only).  Otherwise with the hardware exponential and reciprocal (about 1 ulp each;
// the result is rounded to bf16 right after).
template <bool EXACT> __device__ __forceinline__ float silu_mul(float g, float u) {
  if constexpr (EXACT) return g / (1.0f + expf(-g)) * u;
  return g * u * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
}

// --------------------------------------------------------------------------------------------
// bf16 MFMA kernels
// --------------------------------------------------------------------------------------------
constexpr int BROWS = 256;      // weight rows per block tile
constexpr int BK = BK_ELEMS;    // K elements per stage
constexpr int ROWB = BK * 2;    // bytes per tile row in LDS (eight 16-byte chunks)

// Shapes whose K or N is not a multiple of 64 (RAGGED kernels; both are multiples of 8, so 16-byte
// chunks are valid or invalid as a whole).  The last K stage of a tile holds K % 64 valid elements per row:
// a lane whose chunk lies past them sets the top bit of its offset, which puts the request beyond the
// 2 GiB that the buffer resource admits, and the bounds check of the load unit fills the chunk's LDS
// bytes with zeros for both operands.  Weight rows past N do the same in the even tiles (their row
// groups share one per-lane offset); the ring tiles re-read the last valid row.  The alternative
// these shapes had before, a 64 x 64 fp32-FMA kernel, ran at 50 TFLOP/s (T = 1501, d = 1048, E = 12,
// k = 3, F = 1864: 1.10 ms per layer, now 0.127).
constexpr uint32_t PAST_END = 0x80000000u;
// what a lane that loads chunk `chunk` (0 .. 7) of its rows adds to the offset in the last stage
__device__ __forceinline__ uint32_t ragged_tail(int K, int chunk) {
  const int valid = (K & (BK - 1)) >> 3;          // whole chunks in the last stage (0: all eight)
  return valid != 0 && chunk >= valid ? PAST_END : 0u;
}

// Chunk swizzle of a 128-byte tile row: XOR with the row so that 16 consecutive rows x one
// logical chunk cover a 256-byte bank window exactly once.
__device__ __forceinline__ int swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

template <int N> __device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N <= 63, "vmcnt immediate");
  asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}
// Leaves the requests of the last min(LATER, later) stages (NLOAD per stage) in flight.
template <int LATER, int NLOAD> __device__ __forceinline__ void wait_stages(int later) {
  if constexpr (LATER == 0) {
    wait_vmcnt<0>();
  } else {
    if (later >= LATER) wait_vmcnt<LATER * NLOAD>();
    else wait_stages<LATER - 1, NLOAD>(later);
  }
}

// Barrier at which LDS changes hands: after it, other waves or direct-to-LDS loads overwrite what this
// wave has read, so its reads must have returned (a read still under way when its slot is
// refilled would see the new data).  The wait is stated here and not left to where the compiler puts the reads'
// first use; it costs nothing, as the reads have been consumed by then.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// A wave-uniform value that the optimiser takes for a new one at every call: nothing derived from it is
// computed ahead of a loop and kept.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

// Store of a wave's outputs.  Accumulator (v, lane) holds out[row = m-sub-tile + lane%16]
// [col = n-sub-tile + 4*(lane/16) + v]: 8-byte pieces scattered over 16 rows.  Each wave turns its
// 16-row sub-tile around in a private LDS region (row pitch = row bytes + 32: the 32-byte runs
// that the four lanes of a row write land in 8 banks, and 8 consecutive rows cover all 64) and
// stores whole rows, 16 bytes per lane, so the L2 sees full-line writes.  Starts with a barrier:
// every wave must be done with whatever else the block kept in that LDS.
// MI, NI: accumulator sub-tiles of a wave; WN: waves along the weight rows; the wave's first
// mi_valid sub-tiles are stored, the first one starting at row wave_row0 of the tile.
template <bool GATED, bool EXACT, int MI, int NI, int WN, int NW>
__device__ __forceinline__ void ffn_store_tile(const f32x4_t (&acc)[NI][MI], const TileCoord& tc,
                                               const GemmArgs& p, unsigned char* lds, int wave, int lane,
                                               int mi_valid, int wave_row0) {
  constexpr int NIH = GATED ? NI / 2 : NI;
  const int wn = wave % WN;
  const int l16 = lane & 15;
  const int N = p.N;
  const int n0 = tc.n0;
  lds_barrier();
  constexpr int CW = NIH * 16;                    // output columns of this wave
  constexpr int PITCH = CW * 2 + 32;              // bytes
  constexpr int LPR = CW * 2 / 16;                // lanes that store one row
  constexpr int RPI = 64 / LPR;                   // rows per store instruction
  static_assert((16 % RPI == 0 || RPI == 32) && NW * 16 * PITCH <= 40 * 1024, "staging fits the smallest LDS buffer it is given");
  unsigned char* region = lds + wave * (16 * PITCH);
  bf16_t* out = static_cast<bf16_t*>(p.out);
  const int col0 = n0 + wn * CW;                  // first output column of this wave
  const int32_t* out_map = GATED ? nullptr : p.out_map;   // uniform
  auto mapped_row = [&](int gr) { return min(max(out_map[min(gr, tc.m_end - 1)], 0), p.out_rows - 1); };
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    if (mi < mi_valid) {                          // wave-uniform
      const int row_base = tc.m_begin + wave_row0 + mi * 16;
      // this lane's accumulators belong to row lane%16 of the sub-tile
      const float scale = out_map ? p.out_scale[mapped_row(row_base + l16)] : 1.f;
#pragma unroll
      for (int ni = 0; ni < NIH; ++ni) {
        float o[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (GATED)
            o[u] = silu_mul<EXACT>(acc[ni][mi][u], acc[GATED ? ni + NIH : ni][mi][u]);
          else
            o[u] = out_map ? acc[ni][mi][u] * scale : acc[ni][mi][u];
        }
        const int c = ni * 16 + 4 * (lane >> 4);
        *reinterpret_cast<uint2*>(region + l16 * PITCH + c * 2) =
            make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // same wave: writes land before the reads
#pragma unroll
      for (int it = 0; it < (16 + RPI - 1) / RPI; ++it) {
        const int r = it * RPI + lane / LPR;
        if (RPI > 16 && r >= 16) continue;        // a sub-tile narrower than the wave's store
        const int c = (lane % LPR) * 8;           // first column of this lane's 16 bytes
        const uint4 v = *reinterpret_cast<const uint4*>(region + r * PITCH + c * 2);
        const int gr = row_base + r;
        if (gr < tc.m_end && col0 + c < N) {
          const int dst = out_map ? mapped_row(gr) : gr;
          *reinterpret_cast<uint4*>(out + static_cast<int64_t>(dst) * N + col0 + c) = v;
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // reads done before the region is reused
    }
  }
}

// A part of a split tile leaves its accumulators in its workspace slot, thread-major so that a
// thread's 16 bytes sit next to its neighbours'; the summing launch reads them back the same way.
template <int MI, int NI, int NT>
__device__ __forceinline__ void ffn_store_part(const f32x4_t (&acc)[NI][MI], const TileCoord& tc,
                                               const GemmArgs& p) {
  static_assert(NI * MI * NT * 4 <= SPLIT_SLOT_FLOATS, "slot size");
  float* mine = p.split_ws + static_cast<int64_t>(tc.pslot) * SPLIT_SLOT_FLOATS;
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
      *reinterpret_cast<f32x4_t*>(mine + ((ni * MI + mi) * NT + static_cast<int>(threadIdx.x)) * 4) =
          acc[ni][mi];
}
template <int MI, int NI, int NT>
__device__ __forceinline__ void ffn_sum_parts(f32x4_t (&acc)[NI][MI], const TileCoord& tc,
                                              const GemmArgs& p) {
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const float* first = p.split_ws + static_cast<int64_t>(tc.pslot) * SPLIT_SLOT_FLOATS;
  for (int q = 0; q < tc.nparts; ++q) {           // in part order: the sum does not depend on scheduling
    const float* src = first + static_cast<int64_t>(q) * SPLIT_SLOT_FLOATS;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(
            src + ((ni * MI + mi) * NT + static_cast<int>(threadIdx.x)) * 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[ni][mi][u] += v[u];
      }
  }
}

// --------------------------------------------------------------------------------------------
// Ring tiles: BM x WROWS block tile, WM x WN waves, NSTAGE LDS stages of 64 K-elements with
// NSTAGE - 1 stages of loads in flight.  Bound by the weight stream from HBM: what counts is the bytes
// a CU keeps in flight (64 x 256 tiles: 96 KiB of weights) and that every CU has a tile.  The
// pieces of a last round are 64 x 64 (nine stages), 64 x 128 (six) and 128 x 128 (five), the
// deepest rings that fit.  (Measured, pieces against whole tiles, or 64-row pieces for the 128-row ones:
// down-projection of the Mixtral shape, 128 tiles of K = 14336, at 300 tokens 242 -> 186 us, at
// one token, 32 tiles, 154 -> 73 us.)  SPLIT: tiles of the last round may be cut along K
// instead (see decode_tile): a part leaves its fp32 accumulators in the workspace, and the next launch
// on the stream adds the parts and stores the tile.
// --------------------------------------------------------------------------------------------
constexpr int ffn_ring_lds_bytes(int bm, int wrows, int nstage) { return nstage * (bm + wrows) * ROWB; }

template <int BM, int WROWS, bool GATED, int WM, int WN, int NSTAGE, bool SPLIT, bool WNT, bool RAGGED>
__device__ __forceinline__ void ffn_ring_tile(const GemmArgs& p, const TileCoord& tc, unsigned char* lds) {
  constexpr int NW = WM * WN;                     // waves per block
  constexpr int KSTEPS = BK / 32;                 // MFMA k-steps per stage
  constexpr int MI = BM / WM / 16;                // 16-row activation sub-tiles per wave
  constexpr int NI = WROWS / WN / 16;             // 16-row weight sub-tiles per wave
  constexpr int NIH = GATED ? NI / 2 : NI;        // gated: sub-tiles per weight matrix
  constexpr int WHALF = GATED ? WROWS / 2 : WROWS;  // weight rows per matrix
  constexpr int STAGE = (BM + WROWS) * ROWB;      // bytes per stage
  constexpr int NLOAD = (BM + WROWS) / 8 / NW;    // direct-to-LDS instructions per wave per stage
  constexpr int NLA = BM / 8 / NW;                // ... of which load activation rows
  constexpr int NLB = WHALF / 8 / NW;             // ... of each weight matrix
  constexpr bool MIXED = GATED && NLB == 0;       // one instruction loads both: half the waves each
  static_assert(NLA * 8 * NW == BM && (NLOAD - NLA) * 8 * NW == WROWS && MI >= 1 && NIH >= 1, "tile shape");
  static_assert(NSTAGE > 2, "a ring keeps at least two stages of loads in flight");

  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE);
  const int wm = wave / WN, wn = wave % WN;
  const int K = p.K, N = p.N;
  int kt_first = 0, kt_count = RAGGED ? (K + BK - 1) / BK : K / BK;   // this block's K stages
  if (SPLIT && tc.nparts > 1) {
    kt_first = tc.part * kt_count / tc.nparts;
    kt_count = (tc.part + 1) * kt_count / tc.nparts - kt_first;
  }
  const int KT = kt_count;
  const int n0 = tc.n0;
  const bf16_t* A = static_cast<const bf16_t*>(p.a);
  const bf16_t* B0 = static_cast<const bf16_t*>(p.b0) + static_cast<int64_t>(tc.e) * N * K;
  const bf16_t* B1 = GATED ? static_cast<const bf16_t*>(p.b1) + static_cast<int64_t>(tc.e) * N * K
                           : nullptr;
  // 16-row activation sub-tiles of this wave that hold at least one valid row
  const int rows_valid = min(tc.m_end - tc.m_begin, BM);
  const int mi_valid = max(0, min(MI, (rows_valid - wm * (BM / WM) + 15) / 16));

  // ---- global -> LDS assignment: instruction i of this wave fills row group g = i*NW + wave
  //      (8 rows x 8 chunks = 1 KiB).  Which matrix a row group belongs to depends on i alone,
  //      so each instruction has a uniform 64-bit base and a 32-bit per-lane offset.  Rows past
  //      the end of the segment (or of the weight matrix) re-read the last valid row.
  const bool gathered = p.src_assign != nullptr;  // uniform
  const int k_first = kt_first * BK;              // first K element of this block
  const unsigned char* base_a = reinterpret_cast<const unsigned char*>(
      (gathered ? A : A + static_cast<int64_t>(tc.m_begin) * K) + k_first);
  const unsigned char* base_b0 =
      reinterpret_cast<const unsigned char*>(B0 + static_cast<int64_t>(n0) * K + k_first);
  const unsigned char* base_b1 =
      GATED ? reinterpret_cast<const unsigned char*>(B1 + static_cast<int64_t>(n0) * K + k_first)
            : nullptr;
  uint32_t soff[NLOAD];
#pragma unroll
  for (int i = 0; i < NLOAD; ++i) {
    const int g = i * NW + wave;
    const int row = g * 8 + (lane >> 3);          // row in the stage: [0,BM) x rows, then weights
    const int chunk = (lane & 7) ^ swz(row);      // the chunk of the row this lane fetches
    int r;                                        // row relative to the instruction's base
    if (i < NLA) {
      r = min(row, rows_valid - 1);
      // gathered: the offset is taken from the start of `a` (the host checks that it fits 31 bits)
      if (gathered) r = a_row_of(p, tc.m_begin + r);
    } else {
      const int br = row - BM;
      r = min(br & (WHALF - 1), N - 1 - n0);
    }
    soff[i] = static_cast<uint32_t>(r) * static_cast<uint32_t>(K) * 2u + static_cast<uint32_t>(chunk) * 16u;
  }
  // buffer resources (raw, stride 0) based at the first row of each operand of this tile: the
  // per-lane 32-bit offset and a scalar K offset replace 64-bit per-lane address arithmetic
  const __amdgpu_buffer_rsrc_t rs_a =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base_a), 0, 0x7FFFFFFF, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_b0 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(MIXED && wave >= NW / 2 ? base_b1 : base_b0), 0, 0x7FFFFFFF, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_b1 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(GATED ? base_b1 : base_b0), 0, 0x7FFFFFFF, 0x00020000);
  // The weight rows of an expert that is this one tile are read once by the whole chip: requested
  // with the non-temporal hint they do not displace what other blocks still share in the L2.
  // (Measured with the hint on every ring tile: decode-shaped layer 0.79 -> 0.72 ms, Mixtral shape
  // at 16 tokens 0.51 -> 0.48 ms, its weights then stream at 5.9 TB/s; with two tiles per expert,
  // Mixtral shape at 256 and 448 tokens, 1 to 5 % slower, hence the condition.)
  const bool wgt_nt = WNT && tc.sharers <= 1;   // block-uniform
  static_assert(!RAGGED || NW % 2 == 0, "one K chunk per lane in every load");
  const uint32_t tail = RAGGED ? ragged_tail(K, (lane & 7) ^ swz(wave * 8 + (lane >> 3))) : 0u;
  // instruction i of stage kt into LDS stage `stage` (1 KiB per wave instruction)
  auto issue_load = [&](int i, int kt, int stage) {
    const __amdgpu_buffer_rsrc_t rs = (i < NLA) ? rs_a : (!GATED || MIXED || i < NLA + NLB) ? rs_b0 : rs_b1;
    const uint32_t off = RAGGED && kt == KT - 1 ? soff[i] | tail : soff[i];
    if (i < NLA || !wgt_nt)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (__attribute__((address_space(3))) void*)(lds + stage * STAGE + (i * NW + wave) * 1024), 16,
          static_cast<int>(off), kt * ROWB, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (__attribute__((address_space(3))) void*)(lds + stage * STAGE + (i * NW + wave) * 1024), 16,
          static_cast<int>(off), kt * ROWB, 0, 2);                 // aux bit 1: nt
  };

  // ---- LDS read addresses of the MFMA fragments ------------------------------------------------
  // A lane holds, for row lane%16 of a 16-row sub-tile, the 8 K-elements of one 16-byte chunk of
  // the k-step's four.  Which chunk goes to which lane group is free as long as both operands
  // agree (it only permutes the K order inside the MFMA).  The LDS serves a 16-byte read in
  // passes of lanes {0-7, 32-39}, {8-15, 40-47}, ...: lane groups 0 and 2 therefore take chunks
  // that differ in bit 0 (0 and 1; groups 1 and 3 take 2 and 3), which with the row swizzle
  // makes every pass touch each bank once.
  const int l16 = lane & 15;
  const int f = swz(l16);                         // sub-tile bases are multiples of 16 rows
  const int kgrp = ((lane >> 4) & 1) * 2 + (lane >> 5);
  int koff[KSTEPS];
#pragma unroll
  for (int kk = 0; kk < KSTEPS; ++kk) koff[kk] = (((kk * 4 + kgrp) ^ f) << 4);
  const int x_base = (wm * (BM / WM) + l16) * ROWB;
  // first weight row of sub-tile ni relative to the wave's own first weight row
  auto w_sub = [](int ni) { return GATED ? (ni / NIH) * WHALF + (ni % NIH) * 16 : ni * 16; };
  const int w_base = (BM + (GATED ? wn * (NIH * 16) : wn * (NI * 16)) + l16) * ROWB;

  f32x4_t acc[NI][MI];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int stage) {                 // compiler-scheduled
    const unsigned char* s = lds + stage * STAGE;
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
      bf16x8_t xf[MI], wf[NI];
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
        if (mi < mi_valid)
          xf[mi] = *reinterpret_cast<const bf16x8_t*>(s + x_base + mi * 16 * ROWB + koff[kk]);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        wf[ni] = *reinterpret_cast<const bf16x8_t*>(s + w_base + w_sub(ni) * ROWB + koff[kk]);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
          if (mi < mi_valid)
            acc[ni][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ni], xf[mi], acc[ni][mi], 0, 0, 0);
    }
  };

  // ---- ring pipeline: the loads of stage kt+DIST are issued at the start of stage kt -----------
  constexpr int DIST = NSTAGE - 1;
#pragma unroll
  for (int s = 0; s < DIST; ++s)
    if (s < KT) {
#pragma unroll
      for (int i = 0; i < NLOAD; ++i) issue_load(i, s, s);
    }
  int cur = 0, fill = DIST;                       // slots of stage kt and of stage kt + DIST
  for (int kt = 0; kt < KT; ++kt) {
    // the loads of stage kt are the oldest outstanding; up to DIST-1 later stages may follow
    wait_stages<DIST - 1, NLOAD>(KT - 1 - kt);
    lds_barrier();                    // stage kt landed for all waves; the slot of kt-1 is free
    if (kt + DIST < KT) {
#pragma unroll
      for (int i = 0; i < NLOAD; ++i) issue_load(i, kt + DIST, fill);
    }
    if (mi_valid > 0) compute(cur);
    cur = cur + 1 == NSTAGE ? 0 : cur + 1;
    fill = fill + 1 == NSTAGE ? 0 : fill + 1;
  }

  if (SPLIT && tc.nparts > 1) {
    ffn_store_part<MI, NI, NW * MOE_WAVE>(acc, tc, p);
    return;
  }
  ffn_store_tile<GATED, RAGGED, MI, NI, WN, NW>(acc, tc, p, lds, wave, lane, mi_valid, wm * (BM / WM));
}

// Adds the parts of a split ring tile and stores it.
template <int BM, bool GATED, int WM, int WN>
__device__ __forceinline__ void ffn_ring_sum_tile(const GemmArgs& p, const TileCoord& tc, unsigned char* lds) {
  constexpr int NW = WM * WN;
  constexpr int MI = BM / WM / 16;
  constexpr int NI = BROWS / WN / 16;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE);
  const int wm = wave / WN;
  const int rows_valid = min(tc.m_end - tc.m_begin, BM);
  const int mi_valid = max(0, min(MI, (rows_valid - wm * (BM / WM) + 15) / 16));
  f32x4_t acc[NI][MI];
  ffn_sum_parts<MI, NI, NW * MOE_WAVE>(acc, tc, p);
  ffn_store_tile<GATED, false, MI, NI, WN, NW>(acc, tc, p, lds, wave, lane, mi_valid, wm * (BM / WM));
}

// --------------------------------------------------------------------------------------------
// Even tiles: an expert's c rows are cut into tiles of (nearly) equal height, a
// multiple of 16 rows each, so no segment leaves a small remainder that would have to stream the
// expert's weights once more for a handful of rows: the Mixtral-shaped batch (about 1024 rows
// per expert) runs as four tiles of 256 or 272 rows per expert, whatever the counts are.
// Block tile: up to 320 activation rows x 256 weight rows, K step 64, two activation buffers, then
// two to four weight buffers in LDS (activations first, so that a fragment read selects
// their buffer with its 16-bit offset field).
// 8 waves as 4 (rows) x 2 (weight rows); the tile's 16-row sub-tiles are dealt to the four wave
// rows as evenly as possible (each takes MIV = 0 .. 5 of them, the first wave rows one more than
// the last), so a wave holds up to 5 x 8 accumulator tiles.
//
// Per k-step a wave multiplies in two parts so that ONE register set holds the fragments of both
// operands: part 1 takes the first P1 = ceil(MIV / 2) activation sub-tiles against all eight weight
// sub-tiles; part 2 re-reads those P1 activation fragments for the next k-step, multiplies the
// other MIV - P1 sub-tiles, re-reading each weight fragment right after its last use, and re-reads
// the remaining activation fragments at its end.  Every fragment is requested at least 14 MFMAs
// before it is needed.  LDS reads return in order, so "my fragment has landed" is a count of the
// reads issued after it.  Inline asm pins the order; the compiler does not see these LDS reads, so
// it inserts no waits of its own.  A stage's barrier sits between the two parts of its second
// k-step: by then every fragment of the stage is in registers, the stage's buffers take the loads
// of a later stage, and the next stage's, which have landed, are read from.
//
// Who issues the loads.  A wave that issues a burst of direct-to-LDS loads is held at every one of
// them until the address unit takes it, and issues no MFMA meanwhile.  If all eight waves load
// their eighth of a stage right after the barrier, both waves of every SIMD are held at once and
// the matrix pipe idles.  So the waves form two sets of four, {0-3} and {4-7} (waves w and w + 4 share
// a SIMD), that take turns: set (stage & 1) issues the whole stage while the other set goes
// straight on with its MFMAs, so every SIMD always has a wave that multiplies.  Measured on the
// Mixtral shape: up-projection 6 % faster than with every wave loading; llama4 shape (one tile of about 256
// rows per expert), whole layer 1050 -> 1036 us with turns and three weight buffers.  (One set for the weight
// rows and the other for the activation rows: 12 to 20 % slower on tiles of 65 to 128 rows.)
constexpr int EVEN_BM = 320;
constexpr int EVEN_ACT = EVEN_BM * ROWB;                     // one activation buffer
constexpr int EVEN_WGT = BROWS * ROWB;                       // one weight buffer
constexpr int FFN_LDS = ffn_ring_lds_bytes(RING_ROWS, BROWS, 4) > 2 * (EVEN_ACT + EVEN_WGT)
                             ? ffn_ring_lds_bytes(RING_ROWS, BROWS, 4) : 2 * (EVEN_ACT + EVEN_WGT);

// LDS of an even tile: two activation buffers of 64 MI rows and as many weight buffers as fit beside them.
constexpr int even_wgt_buffers(int mi) { return mi <= 2 ? 4 : mi <= 4 ? 3 : 2; }
// How the tile's sub-tiles are dealt to wave row wm (of 4): count and first row.
__device__ __forceinline__ void even_wave_rows(int rows_valid, int wm, int& miv, int& row0) {
  const int nsub = (rows_valid + 15) >> 4;
  const int q = nsub >> 2, r = nsub & 3;
  miv = q + (wm < r ? 1 : 0);
  row0 = 16 * (wm * q + min(wm, r));
}

// MI: 16-row sub-tiles a wave can hold.  MI = 5: tiles of up to 320 rows, two weight buffers (144 KiB).
// MI = 4: tiles of up to 256 rows; the 16 KiB the activation buffers give back make a third weight
// buffer (160 KiB), and the weight rows are requested a stage earlier than the activation rows:
// they are the operand that misses the L2 (an XCD's tiles share activation rows far more often
// than weight rows), so their requests take longest to return.  MI = 2: tiles of up to 128 rows, bound by
// the weight stream; a fourth weight buffer, and with the two sets of waves taking turns a weight
// request has three stage times to return (each set waits for its own requests only, and its next
// ones, whose activation rows are due a stage later, come two stages on).
// (Measured against two or more 64-row ring tiles per expert, up-projection: Mixtral shape at 500
// tokens 512 -> 350 us, 5.4 TB/s of weights, phi shape at 600 tokens 385 -> 313 us, 64-expert shape at 1024
// tokens 186 -> 148 us.)
template <bool GATED, bool SPLIT, bool WNT, bool RAGGED, int MI>
__device__ __forceinline__ void ffn_even_tile(const GemmArgs& p, const TileCoord& tc, unsigned char* lds) {
  constexpr int NW = 8, WN = 2;
  constexpr int BM = MI * 64, NI = 8;
  constexpr int NIH = GATED ? NI / 2 : NI;
  constexpr int NLA = BM / 8 / 4;                 // up to 10 activation row groups per loading wave and stage
  constexpr int ACT = BM * ROWB;                  // one activation buffer
  constexpr int NWB = even_wgt_buffers(MI);
  constexpr int W_BASE = 2 * ACT;                 // LDS offset of the weight buffers
  static_assert(MI == 2 || MI == 4 || MI == 5, "wave tile");
  static_assert(W_BASE + NWB * EVEN_WGT <= FFN_LDS, "LDS budget");

  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE);
  const int wm = wave / WN, wn = wave % WN;
  constexpr int ns = 4;                           // waves that share a stage's loads
  const int lw = wave & 3;                        // this wave's place among them
  const int lset = wave >> 2;                     // ... and the stages it loads: stage & 1 == lset
  const int K = p.K, N = p.N;
  int KT = RAGGED ? (K + BK - 1) / BK : K / BK, k_first = 0;   // this block's K stages
  if (SPLIT && tc.nparts > 1) {
    const int kt_first = tc.part * KT / tc.nparts;
    KT = (tc.part + 1) * KT / tc.nparts - kt_first;
    k_first = kt_first * BK;
  }
  const int n0 = tc.n0;
  const int rows_valid = min(tc.m_end - tc.m_begin, BM);
  int miv, row0;
  even_wave_rows(rows_valid, wm, miv, row0);

  // ---- global -> LDS.  A wave instruction fills an 8-row group of 1 KiB.  A loading wave takes
  //      activation groups i * ns + lw (only those that hold a valid row) and weight groups
  //      i * ns + lw (N - n0 is a multiple of 64, RAGGED: of 8, so a group is inside the weight
  //      matrix or outside as a whole).  The rows of a wave's weight groups are multiples of
  //      32 rows apart (same swizzle): one per-lane offset, the rest is a scalar.  Activation rows
  //      past the end of the segment re-read its last row.
  const bool gathered = p.src_assign != nullptr;
  const bf16_t* A = static_cast<const bf16_t*>(p.a) + k_first;
  const bf16_t* B0 = static_cast<const bf16_t*>(p.b0) + static_cast<int64_t>(tc.e) * N * K + k_first;
  const bf16_t* B1 =
      GATED ? static_cast<const bf16_t*>(p.b1) + static_cast<int64_t>(tc.e) * N * K + k_first : B0;
  // buffer resources (raw, stride 0) based at the first row of each operand of this tile: the
  // per-lane 32-bit offset and a scalar offset replace 64-bit per-lane address arithmetic
  // (gathered rows: the offset is taken from the start of `a`; the host checks that it fits 31 bits)
  const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(gathered ? A : A + static_cast<int64_t>(tc.m_begin) * K), 0, 0x7FFFFFFF, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_b0 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(B0 + static_cast<int64_t>(n0) * K), 0, 0x7FFFFFFF, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_b1 = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(B1 + static_cast<int64_t>(n0) * K), 0, 0x7FFFFFFF, 0x00020000);
  const int n_act = min(BM / 8 / ns, max(0, (((rows_valid + 7) >> 3) - lw + ns - 1) / ns));
  const int w_rows = min(GATED ? 128 : 256, N - n0);          // weight rows of this tile per matrix
  uint32_t soff_a[NLA], soff_w;
  {
    const int br = lw * 8 + (lane >> 3);
    const int chunk = (lane & 7) ^ swz(br);
    soff_w = static_cast<uint32_t>(br) * static_cast<uint32_t>(K) * 2u + static_cast<uint32_t>(chunk) * 16u;
  }
  // (the row groups a lane loads, of either operand, are an even number of groups apart: one chunk)
  const uint32_t tail = RAGGED ? ragged_tail(K, (lane & 7) ^ swz(lw * 8 + (lane >> 3))) : 0u;
  // The activation rows of stage kt go to activation buffer kt % 2 and are requested two stages
  // ahead, the weight rows to weight buffer kt % NWB, NWB stages ahead.  The requests made after the
  // barrier of stage j (activations of j + 2, then weights of j + NWB) all come from wave set j & 1.
  // What the requests of a stage have in common is computed from `fresh` values: the optimiser would
  // otherwise carry an LDS address and a condition mask per request, and a product per row group, through the
  // K loop, more than there are scalar registers, and fetch them back lane by lane (10 to 34 such reads
  // per two stages; measured without them, whole layer: 128-expert step of 8 to 32 tokens 1 to 2 %,
  // Mixtral shape at 2000 tokens 1 %, llama4 shape at 4096 tokens 0.6 % faster).
  auto issue_act = [&](int kt) {
    if (lset != (kt & 1)) return;
    const uint32_t past = RAGGED && kt == KT - 1 ? tail : 0u;
    const int n = fresh(n_act), to = fresh((kt & 1) * ACT + lw * 1024);
#pragma unroll
    for (int i = 0; i < NLA; ++i)
      if (i < n)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rs_a, (__attribute__((address_space(3))) void*)(lds + to + i * ns * 1024), 16,
            static_cast<int>(RAGGED ? soff_a[i] | past : soff_a[i]), kt * ROWB, 0, 0);
  };
  // Every wave makes the same number of weight requests per stage (W_LOADS), so that a wait can
  // leave exactly one stage's weight requests outstanding: a group outside the weight matrix (the
  // last n-tile of a matrix whose row count is not a multiple of the tile) re-reads the last groups
  // inside, or, RAGGED, asks beyond the resource; its products are never stored.
  constexpr int W_LOADS = 32 / ns;
  // WNT: weight rows that at most two tiles read (an expert of one or two tiles) are requested with
  // the non-temporal hint: nothing will ask for them again, and they stop displacing the activation
  // rows, which the other n-tiles of the round and the later rounds re-read, from the L2.  Weight
  // rows shared by more tiles keep the default policy (measured with the hint on every tile: the
  // Mixtral shape, four tiles per expert, up-projection 4 % slower; llama4 and phi shapes, one and
  // two tiles per expert, both GEMMs 4 to 7 % faster).  The branch per stage costs a launch whose
  // tiles all keep the default policy about 1 %, so the host builds it in (WNT) only for calls with
  // few rows per expert.
  const bool wgt_nt = WNT && tc.sharers <= WGT_NT_MAX_SHARERS;       // block-uniform
  auto issue_wgt_with = [&](int kt, int wb, auto aux_c) {
    constexpr int AUX = decltype(aux_c)::value;
    const uint32_t base = RAGGED && kt == KT - 1 ? soff_w | tail : soff_w;
    const int to = fresh(W_BASE + wb * EVEN_WGT + lw * 1024);
    int at = 0;                                   // scalar offset: the stage's first byte, and the rows before the group
#pragma unroll
    for (int i = 0; i < W_LOADS; ++i) {
      // group i * ns + lw of the 32 weight row groups; gated: groups 0-15 are W1 rows 0-127 of the
      // tile, groups 16-31 the same rows of W3
      const int g0 = i * ns * 8;                  // first row of the step (lw = 0)
      const int jr = GATED ? (g0 & 127) : g0;     // ... inside its matrix
      if (jr == 0) at = kt * ROWB;
      else if (RAGGED || jr < w_rows) at += K * (ns * 8 * 2);
      at = fresh(at);
      uint32_t off = base;                        // RAGGED: the wave's own group of the step may lie past the end
      if (RAGGED && jr + lw * 8 >= w_rows) off |= PAST_END;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          !GATED || g0 < 128 ? rs_b0 : rs_b1, (__attribute__((address_space(3))) void*)(lds + to + i * ns * 1024),
          16, static_cast<int>(off), at, 0, AUX);
    }
  };
  auto issue_wgt = [&](int kt, int wb) {
    if (lset != ((kt + NWB) & 1)) return;
    if (wgt_nt)
      issue_wgt_with(kt, wb, std::integral_constant<int, 2>{});    // aux bit 1: nt
    else
      issue_wgt_with(kt, wb, std::integral_constant<int, 0>{});
  };

  // ---- LDS addresses of this lane's fragments per k-step.  A lane holds, for row lane%16 of a
  //      16-row sub-tile, the 8 K-elements of one 16-byte chunk of the k-step's four.  Which chunk
  //      goes to which lane group is free as long as both operands agree (it only permutes the K
  //      order inside the MFMA).  The LDS serves a 16-byte read in passes of lanes {0-7, 32-39},
  //      {8-15, 40-47}, ...: lane groups 0 and 2 therefore take chunks that differ in bit 0 (0 and
  //      1; groups 1 and 3 take 2 and 3), which with the row swizzle makes every pass touch each
  //      bank once.
  const int l16 = lane & 15;
  const int f = swz(l16);                         // sub-tile bases are multiples of 16 rows
  const int kgrp = ((lane >> 4) & 1) * 2 + (lane >> 5);
  int xa[2], wa[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const int ko = ((kk * 4 + kgrp) ^ f) << 4;
    xa[kk] = (row0 + l16) * ROWB + ko;
    wa[kk] = W_BASE + (wn * (NIH * 16) + l16) * ROWB + ko;
  }

  f32x4_t acc[NI][MI];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = f32x4_t{0.f, 0.f, 0.f, 0.f};

#define MOE_RD(dst, addr, off) \
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "i"(off) : "memory")
#define MOE_MFMA(c, w, x) \
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(w), "v"(x))
#define MOE_X_OFF(buf, mi) ((buf) * ACT + (mi) * 16 * ROWB)
#define MOE_W_OFF(ni) ((GATED ? ((ni) / NIH) * 128 + ((ni) % NIH) * 16 : (ni) * 16) * ROWB)
  static_assert(MOE_W_OFF(NI - 1) < 65536 && MOE_X_OFF(1, MI - 1) < 65536, "ds_read offset field");

  auto k_loop = [&](auto miv_c) {
    constexpr int MIV = decltype(miv_c)::value;
    constexpr int P1 = (MIV + 1) / 2, P2 = MIV - P1;
    bf16x8_t x[MI], w[NI];
    // the fragments of a k-step are always requested in the order x[0..P1), w[0..NI), x[P1..MIV)
    auto part1 = [&]() {
      if constexpr (MIV > 0) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
          asm volatile("s_waitcnt lgkmcnt(%0)" ::"i"(NI - 1 - ni + P2) : "memory");
#pragma unroll
          for (int mi = 0; mi < P1; ++mi) MOE_MFMA(acc[ni][mi], w[ni], x[mi]);
        }
      }
    };
    // kk, buf: the k-step and activation buffer the next fragments come from; wv: this lane's
    // address in the weight buffer they come from
    auto part2 = [&](auto kk_c, auto buf_c, int wv) {
      constexpr int KK = decltype(kk_c)::value, BUF = decltype(buf_c)::value;
      if constexpr (MIV > 0) {
#pragma unroll
        for (int mi = 0; mi < P1; ++mi) MOE_RD(x[mi], xa[KK], MOE_X_OFF(BUF, mi));
        if constexpr (P2 > 0) asm volatile("s_waitcnt lgkmcnt(%0)" ::"i"(P1) : "memory");
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
          for (int mi = P1; mi < MIV; ++mi) MOE_MFMA(acc[ni][mi], w[ni], x[mi]);
          MOE_RD(w[ni], wv, MOE_W_OFF(ni));
        }
#pragma unroll
        for (int mi = P1; mi < MIV; ++mi) MOE_RD(x[mi], xa[KK], MOE_X_OFF(BUF, mi));
      }
    };
    using K0 = std::integral_constant<int, 0>;
    using K1 = std::integral_constant<int, 1>;
    int wb = 0;                                   // weight buffer of the current stage (uniform)
    auto stage = [&](int kt, auto par_c) {
      constexpr int PAR = decltype(par_c)::value;
      const int wb_next = wb + 1 == NWB ? 0 : wb + 1;
      part1();
      part2(K1{}, std::integral_constant<int, PAR>{}, wa[1] + wb * EVEN_WGT);
      part1();
      // Stage kt + 1 must have landed.  Requests return in order, and the last ones of the set whose turn
      // it was after the barrier of stage kt - 1 are the activation rows of kt + 1, then the weight
      // rows of kt - 1 + NWB: with three buffers or more those may stay in flight.  The last ones of the
      // other set are a stage older: weight rows of kt - 2 + NWB, which four buffers spare too.
      const bool turn = lset == ((kt - 1) & 1);
      bool spare = false;
      if constexpr (NWB == 3) spare = kt >= 1 && kt + 2 < KT && turn;
      if constexpr (NWB == 4) spare = kt + (turn ? 3 : 2) < KT;
      if (NWB >= 3 && spare)
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"i"(W_LOADS) : "memory");
      else
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (kt + 2 < KT) issue_act(kt + 2);
      if (kt + NWB < KT) issue_wgt(kt + NWB, wb);
      // (after the tile's last stage these reads return whatever the buffer holds and go unused)
      part2(K0{}, std::integral_constant<int, PAR ^ 1>{}, wa[0] + wb_next * EVEN_WGT);
      wb = wb_next;
    };
    if constexpr (MIV > 0) {
#pragma unroll
      for (int mi = 0; mi < P1; ++mi) MOE_RD(x[mi], xa[0], MOE_X_OFF(0, mi));
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) MOE_RD(w[ni], wa[0], MOE_W_OFF(ni));
#pragma unroll
      for (int mi = P1; mi < MIV; ++mi) MOE_RD(x[mi], xa[0], MOE_X_OFF(0, mi));
    }
    int kt = 0;
    for (; kt + 2 <= KT; kt += 2) {
      stage(kt, K0{});
      stage(kt + 1, K1{});
    }
    if (kt < KT) stage(kt, K0{});
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the unused reads of the last stage
    // the compiler's hazard handling does not see asm MFMAs: let the last results retire
    // before ordinary VALU code reads the accumulators
    asm volatile("s_nop 15\n s_nop 15\n s_nop 15\n s_nop 15" ::: "memory");
  };

  // prologue: the map entries of a call that reads x through the map are requested first, the weight rows,
  // whose addresses need no memory, while they travel, then the activation rows of stages 0 and 1.
  // With four weight buffers the weight rows of stages 2 and 3 come last and stay in flight over
  // the first barrier, in the order in which the k loop goes on.
#pragma unroll
  for (int i = 0; i < NLA; ++i) {
    const int r = min((i * ns + lw) * 8 + (lane >> 3), rows_valid - 1);
    soff_a[i] = static_cast<uint32_t>(gathered ? p.src_assign[tc.m_begin + r] : r);
  }
#pragma unroll
  for (int s = 0; s < (NWB == 4 ? 2 : NWB); ++s)
    if (s < KT) issue_wgt(s, s);
#pragma unroll
  for (int i = 0; i < NLA; ++i) {
    const int chunk = (lane & 7) ^ swz((i * ns + lw) * 8 + (lane >> 3));   // the chunk of the row this lane fetches
    int r = static_cast<int>(soff_a[i]);
    if (gathered) r = min(max(r / p.k_div, 0), p.a_rows - 1);
    soff_a[i] = static_cast<uint32_t>(r) * static_cast<uint32_t>(K) * 2u + static_cast<uint32_t>(chunk) * 16u;
  }
  issue_act(0);
  if (KT > 1) issue_act(1);
  if (NWB == 4) {
#pragma unroll
    for (int s = 2; s < NWB; ++s)
      if (s < KT) issue_wgt(s, s);
  }
  if (NWB == 4 && KT >= NWB)
    asm volatile("s_waitcnt vmcnt(%0)" ::"i"(W_LOADS) : "memory");
  else
    wait_vmcnt<0>();
  lds_barrier();
  switch (miv) {                                  // wave-uniform
    case 0: k_loop(std::integral_constant<int, 0>{}); break;
    case 1: k_loop(std::integral_constant<int, 1>{}); break;
    case 2: k_loop(std::integral_constant<int, 2>{}); break;
    case 3:
      if constexpr (MI >= 3) k_loop(std::integral_constant<int, 3>{});
      break;
    case 4:
      if constexpr (MI >= 4) k_loop(std::integral_constant<int, 4>{});
      break;
    default:
      if constexpr (MI >= 5) k_loop(std::integral_constant<int, 5>{});
      break;
  }
#undef MOE_RD
#undef MOE_MFMA
#undef MOE_X_OFF
#undef MOE_W_OFF

  if (SPLIT && tc.nparts > 1) {
    ffn_store_part<MI, NI, NW * MOE_WAVE>(acc, tc, p);
    return;
  }
  // the store turns the sub-tiles around in the first 20 (gated) or 36 KiB of the LDS, whatever buffers lie
  // there (every wave has read its last fragments before the store's barrier)
  ffn_store_tile<GATED, RAGGED, MI, NI, WN, NW>(acc, tc, p, lds, wave, lane, miv, row0);
}

// Which pipeline a tile takes: sub-tiles per wave (MI) of the even tile, 0 for a ring tile.
// The more weight buffers the better where the weight rows come from HBM.  Where experts hold several
// tiles each (!WNT), the tiles share them through the L2, and only the down-projection, whose
// reduction is the longer one, gains from the third buffer.  (Measured: Mixtral shape at 192 rows per
// expert, up-projection 434 -> 389 us with three; at 1024 rows 1 % slower, down-projection 4.5 %
// faster; skewed 64-expert layer of 8192 tokens, the cold experts' tiles with four, up-projection
// 1 % slower.)  few_buffers: see launch_bf16.
template <bool GATED, bool WNT> __device__ __forceinline__ int tile_mi(const GemmArgs& p, const TileCoord& tc) {
  const bool three = GATED ? WNT && !(p.few_buffers && tc.sharers > 1) : true;
  return tc.height <= RING_ROWS ? 0 : WNT && tc.height <= 128 ? 2 : three && tc.height <= 256 ? 4 : 5;
}

template <bool GATED, bool SPLIT, bool WNT, bool RAGGED>
__global__ __launch_bounds__(512) void ffn_bf16_kernel(GemmArgs p) {
  extern __shared__ __align__(1024) unsigned char lds[];
  static_assert(ffn_ring_lds_bytes(RING_ROWS, 64, 9) <= FFN_LDS && ffn_ring_lds_bytes(RING_ROWS, 128, 6) <= FFN_LDS &&
                    ffn_ring_lds_bytes(NSPLIT_ROWS, 128, 5) <= FFN_LDS, "pieces' rings fit the launch's LDS");
  TileCoord tc;
  if (!decode_tile<SPLIT, WNT>(p, tc)) return;
  const int rows = tc.m_end - tc.m_begin;         // block-uniform
  if (!SPLIT && tc.n_pieces == 4)
    ffn_ring_tile<RING_ROWS, 64, GATED, 4, 2, 9, false, WNT, RAGGED>(p, tc, lds);
  else if (!SPLIT && tc.n_pieces == 2 && rows <= RING_ROWS)
    ffn_ring_tile<RING_ROWS, 128, GATED, 2, 4, 6, false, WNT, RAGGED>(p, tc, lds);
  else if (!SPLIT && tc.n_pieces == 2)
    ffn_ring_tile<NSPLIT_ROWS, 128, GATED, 2, 4, 5, false, WNT, RAGGED>(p, tc, lds);
  else switch (tile_mi<GATED, WNT>(p, tc)) {
    case 0: ffn_ring_tile<RING_ROWS, BROWS, GATED, 2, 4, 4, SPLIT, WNT, RAGGED>(p, tc, lds); break;
    case 2:
      if constexpr (WNT) ffn_even_tile<GATED, SPLIT, WNT, RAGGED, 2>(p, tc, lds);
      break;
    case 4:
      if constexpr (WNT || !GATED) ffn_even_tile<GATED, SPLIT, WNT, RAGGED, 4>(p, tc, lds);
      break;
    default: ffn_even_tile<GATED, SPLIT, WNT, RAGGED, 5>(p, tc, lds); break;
  }
}

// The launch after ffn_bf16_kernel<.., SPLIT>: adds the parts of every split tile and stores it.
template <bool GATED, int MI>
__device__ __forceinline__ void ffn_even_sum_tile(const GemmArgs& p, const TileCoord& tc, unsigned char* lds) {
  constexpr int NW = 8, WN = 2, NI = 8;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE);
  int miv, row0;
  even_wave_rows(min(tc.m_end - tc.m_begin, MI * 64), wave / WN, miv, row0);
  f32x4_t acc[NI][MI];
  ffn_sum_parts<MI, NI, NW * MOE_WAVE>(acc, tc, p);
  ffn_store_tile<GATED, false, MI, NI, WN, NW>(acc, tc, p, lds, wave, lane, miv, row0);
}
template <bool GATED, bool WNT>
__global__ __launch_bounds__(512) void ffn_bf16_sum_parts_kernel(GemmArgs p) {
  extern __shared__ __align__(1024) unsigned char lds[];
  TileCoord tc;
  if (!decode_tile<true, WNT>(p, tc)) return;
  switch (tile_mi<GATED, WNT>(p, tc)) {
    case 0: ffn_ring_sum_tile<RING_ROWS, GATED, 2, 4>(p, tc, lds); break;
    case 2:
      if constexpr (WNT) ffn_even_sum_tile<GATED, 2>(p, tc, lds);
      break;
    case 4:
      if constexpr (WNT || !GATED) ffn_even_sum_tile<GATED, 4>(p, tc, lds);
      break;
    default: ffn_even_sum_tile<GATED, 5>(p, tc, lds); break;
  }
}

// --------------------------------------------------------------------------------------------
// fp32 layers.  Blocks of 4 waves; each wave takes all the tile's 16-row sub-tiles against its own 16 weight
// rows of each matrix, so the waves are equally busy whatever the row count is.  Segments are cut as for the
// bf16 kernels, in pairs of sub-tiles (singly: no difference at 44 to 250 rows per expert).  K step 32
// (128-byte rows).  Two ways to multiply:
//
// f32_split_tile (33 to 64 rows).  The bf16 matrix instruction is 16 times as fast as the fp32 one.  A value
// is cut into three bf16 pieces, each the rounded rest of the ones before: they hold its 24 bits exactly.  All
// piece products but the smallest (2^-32 of the whole or less) are multiplied.  The matrix instruction does not round its sum
// to nearest, so the leading products have an accumulator of their own and the seven others, 2^-7 of them and less, another;
// the two are added by a rounded addition, per stage (gated) or at the end (ungated: there are registers
// for both).  A wave's weight rows are nobody else's, so they go from memory to registers in fragment order and are cut
// there; the activation rows are cut once per block, by the thread that loads them, and shared through three LDS planes.
// Error against 64-bit sums (2-norm, each GEMM by itself, K = 260 to 2048): 1.7e-7 to 4.7e-7, the fp32 instruction 4.4e-7
// to 1.23e-6.  A sum of one product: within 1.0002 x 2^-24 of it, 0.15 % not the nearest fp32 number (six products in one
// accumulator: 2.4 x 2^-24 and 19 %).
// Bound by the matrix pipe and the vector instructions of the cutting, which overlap only between waves:
// three or four blocks per CU and few registers (four blocks in a wave of 128 registers spill; two with
// stage s + 1 cut ahead between the MFMAs of stage s: 5 to 10 % slower; rows of both operands through LDS: 10 %;
// 128-row tiles 5 % faster at 2000 tokens, 10 % slower at 1000).
//
// f32_exact_rows (up to 32 rows).  v_mfma_f32_16x16x4_f32.  Few rows wait for their weights, and cutting them
// would lengthen every stage's chain of load, cut, multiply (60 tokens of the shape below 94 -> 117 us).
// Two stages for the gated tiles (three: 11 % slower, a block per CU less).
//
// (d = 1024, E = 16, k = 2, F = 2048, fp32 instruction alone -> now, us: 1000 tokens, up 151 -> 140, down 98 -> 87, 115 TFLOP/s;
// both GEMMs of 2000 tokens 436 -> 387; d = 1280, E = 4, k = 1, F = 2400, 2000 tokens 331 -> 289.  Six products in one
// accumulator of unscaled pieces: 121 and 77, 335, 242.)
// --------------------------------------------------------------------------------------------
constexpr int F32_NW = 4, F32_BN = 64, F32_BK = 32, F32_BM = 64, F32_EXACT_ROWS = 32;
constexpr int F32_PROW = F32_BK * 2;              // bytes of a row in a plane
constexpr int F32_PLANE = F32_BM * F32_PROW;
constexpr int f32_stages(bool gated) { return gated ? 2 : 3; }
constexpr int ffn_f32_lds_bytes(bool gated) {
  const int exact = f32_stages(gated) * (F32_EXACT_ROWS + (gated ? 2 : 1) * F32_BN) * ROWB, split = 2 * 3 * F32_PLANE;
  return exact > split ? exact : split;
}

// Buffer resources of a tile's operands (see the bf16 kernels).
struct F32Operands {
  __amdgpu_buffer_rsrc_t a, b0, b1;
};
template <bool GATED>
__device__ __forceinline__ F32Operands f32_operands(const GemmArgs& p, const TileCoord& tc, int m_first) {
  const float* A = static_cast<const float*>(p.a) + (p.src_assign ? 0 : static_cast<int64_t>(m_first) * p.K);
  const int64_t b_off = (static_cast<int64_t>(tc.e) * p.N + tc.n0) * p.K;
  const float* B0 = static_cast<const float*>(p.b0) + b_off;
  const float* B1 = GATED ? static_cast<const float*>(p.b1) + b_off : B0;
  return {__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(A), 0, 0x7FFFFFFF, 0x00020000),
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(B0), 0, 0x7FFFFFFF, 0x00020000),
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(B1), 0, 0x7FFFFFFF, 0x00020000)};
}

// Accumulator (v, lane) is row lane % 16 of the sub-tile, columns 4 (lane / 16) .. + 3 of the wave's 16; it holds
// 1 / UNIT of the product.
template <bool GATED, int MI>
__device__ __forceinline__ void f32_store(const f32x4_t (&acc)[GATED ? 2 : 1][MI], const GemmArgs& p, int n0, int m_first,
                                          int m_end, const float UNIT = 1.f) {
  const int lane = lane_id(), wave = threadIdx.x / MOE_WAVE;
  float* out = static_cast<float*>(p.out);
  const int c = n0 + wave * 16 + 4 * (lane >> 4);
  const int32_t* out_map = GATED ? nullptr : p.out_map;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    int gr = m_first + mi * 16 + (lane & 15);
    if (gr >= m_end || c >= p.N) continue;        // (N is a multiple of 4)
    float scale = 1.f;
    if (out_map) {
      gr = min(max(out_map[gr], 0), p.out_rows - 1);
      scale = p.out_scale[gr];
    }
    f32x4_t o;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float v = acc[0][mi][u] * UNIT;
      o[u] = GATED ? silu_mul<true>(v, acc[GATED ? 1 : 0][mi][u] * UNIT) : out_map ? v * scale : v;
    }
    *reinterpret_cast<f32x4_t*>(out + static_cast<int64_t>(gr) * p.N + c) = o;
  }
}

// Rows m_first .. m_end - 1 (at most 32) of the tile on the fp32 matrix instruction.  Tile rows in LDS as in
// the bf16 kernels (same swizzle and chunk order; a chunk is four k-values, one per instruction).
template <bool GATED>
__device__ __forceinline__ void f32_exact_rows(const GemmArgs& p, const TileCoord& tc, unsigned char* lds, int m_first,
                                               int m_end) {
  constexpr int NMAT = GATED ? 2 : 1, BM = F32_EXACT_ROWS;
  constexpr int NSTAGE = f32_stages(GATED);
  constexpr int STAGE = (BM + NMAT * F32_BN) * ROWB;
  constexpr int NLA = BM / 8 / F32_NW, NLB = F32_BN / 8 / F32_NW, NLOAD = NLA + NMAT * NLB;
  constexpr int MI = BM / 16;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE);
  const int K = p.K, N = p.N, KT = (K + F32_BK - 1) / F32_BK;
  const int n0 = tc.n0;
  const int rows_valid = min(m_end - m_first, BM);
  const F32Operands rs = f32_operands<GATED>(p, tc, m_first);
  // instruction i of a wave fills 8-row group i * 4 + wave of the stage: activation rows, then the rows
  // of W1 (or W2), then of W3; rows past the end re-read the last valid one; chunks past K in the
  // last stage come out as zeros (see ragged_tail)
  const int chunk = (lane & 7) ^ swz(wave * 8 + (lane >> 3));
  uint32_t soff[NLOAD];
#pragma unroll
  for (int i = 0; i < NLOAD; ++i) {
    const int row = (i * F32_NW + wave) * 8 + (lane >> 3);
    int r;
    if (i < NLA) {
      r = min(row, rows_valid - 1);
      if (p.src_assign) r = a_row_of(p, m_first + r);
    } else {
      r = min((row - BM) & (F32_BN - 1), N - 1 - n0);
    }
    soff[i] = static_cast<uint32_t>(r) * static_cast<uint32_t>(K) * 4u + static_cast<uint32_t>(chunk) * 16u;
  }
  const int tail_chunks = (K & (F32_BK - 1)) >> 2;
  const uint32_t tail = tail_chunks != 0 && chunk >= tail_chunks ? PAST_END : 0u;
  auto issue = [&](int kt, int stage) {
    const uint32_t past = kt == KT - 1 ? tail : 0u;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          i < NLA ? rs.a : i < NLA + NLB ? rs.b0 : rs.b1,
          (__attribute__((address_space(3))) void*)(lds + stage * STAGE + (i * F32_NW + wave) * 1024), 16,
          static_cast<int>(soff[i] | past), kt * ROWB, 0, 0);
  };
  const int l16 = lane & 15, f = swz(l16), kgrp = ((lane >> 4) & 1) * 2 + (lane >> 5);
  int koff[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) koff[kk] = ((kk * 4 + kgrp) ^ f) << 4;
  const int x_base = l16 * ROWB;
  const int w_base = (BM + wave * 16 + l16) * ROWB;
  f32x4_t acc[NMAT][MI];
#pragma unroll
  for (int m = 0; m < NMAT; ++m)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) acc[m][mi] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  constexpr int DIST = NSTAGE - 1;
#pragma unroll
  for (int s = 0; s < DIST; ++s)
    if (s < KT) issue(s, s);
  auto k_loop = [&](auto miv_c) {
    constexpr int MIV = decltype(miv_c)::value;
    for (int kt = 0; kt < KT; ++kt) {
      const int later = min(DIST - 1, KT - 1 - kt);
      if (later >= 1) wait_vmcnt<NLOAD>();
      else wait_vmcnt<0>();
      lds_barrier();
      if (kt + DIST < KT) issue(kt + DIST, (kt + DIST) % NSTAGE);
      const unsigned char* s = lds + (kt % NSTAGE) * STAGE;
      f32x4_t xf[2][MIV], wf[2][NMAT];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int m = 0; m < NMAT; ++m)
          wf[kk][m] = *reinterpret_cast<const f32x4_t*>(s + w_base + m * (F32_BN * ROWB) + koff[kk]);
#pragma unroll
        for (int mi = 0; mi < MIV; ++mi)
          xf[kk][mi] = *reinterpret_cast<const f32x4_t*>(s + x_base + mi * 16 * ROWB + koff[kk]);
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int m = 0; m < NMAT; ++m)
#pragma unroll
            for (int mi = 0; mi < MIV; ++mi)
              acc[m][mi] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[kk][m][u], xf[kk][mi][u], acc[m][mi], 0, 0, 0);
    }
  };
  static_assert(MI == 2 && DIST <= 2, "cases below and waits above");
  if (rows_valid <= 16) k_loop(std::integral_constant<int, 1>{});     // block-uniform
  else k_loop(std::integral_constant<int, 2>{});
  f32_store<GATED, MI>(acc, p, n0, m_first, m_end);
}

// Values are cut at F32_SCALE times their size: the pieces of every normal fp32 value are then normal bf16 values, and
// no bit of a product that fp32 can hold falls below the range, whatever else its row holds.  At the upper end
// a value of 2^104 and more, or products that add up to 2^80, give an infinite piece or sum, and an infinity stays
// one or turns into a NaN: see f32_split_tile.
constexpr float F32_SCALE = 0x1p24f, F32_UNSCALE = 0x1p-48f;

// Four values to four bf16 of each of the three planes (exact: 8 + 8 + 8 bits and the signs of the rests).
__device__ __forceinline__ void f32_split(f32x4_t r, uint2 (&q)[3]) {
  r *= F32_SCALE;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    q[i] = make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
    if (i < 2) r = f32x4_t{r[0] - bf16lo(q[i].x), r[1] - bf16hi(q[i].x), r[2] - bf16lo(q[i].y), r[3] - bf16hi(q[i].y)};
  }
}
// Chunk swizzle of a 64-byte plane row: 8 rows x the two chunks of an LDS pass cover each bank once.
__device__ __forceinline__ int swz64(int row) { return (row >> 1) & 2; }

// Returns false, and stores nothing, if a sum is not finite (block-uniform): the operands may have left the pieces'
// range, which costs such a tile twice its time and more (2000 tokens of d = 1024, F = 2048 that all hit it in the
// down-projection: 324 us, 155 if none does, 162 by the fp32 instruction alone).
template <bool GATED>
__device__ __forceinline__ bool f32_split_tile(const GemmArgs& p, const TileCoord& tc, unsigned char* lds) {
  constexpr int NMAT = GATED ? 2 : 1, BM = F32_BM;
  constexpr int NLA = BM / 32, MI = BM / 16;
  constexpr int STAGE = 3 * F32_PLANE;
  const int lane = lane_id(), tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE);
  const int K = p.K, N = p.N, KT = (K + F32_BK - 1) / F32_BK;
  const int n0 = tc.n0;
  const int rows_valid = min(tc.m_end - tc.m_begin, BM);
  const F32Operands rs = f32_operands<GATED>(p, tc, tc.m_begin);
  // activations: thread (row tid / 8 + 32 i, chunk tid % 8 of 16 bytes); weights: lane (row lane % 16 of the wave's,
  // chunks lane / 16 and lane / 16 + 4, the k-values of its MFMA fragment).  Rows past the end re-read the
  // last valid one; chunks past K, and stages past the last, come out as zeros.
  const int l16 = lane & 15, kg = lane >> 4, chunk = tid & 7;
  uint32_t soff_a[NLA], soff_w[2];
#pragma unroll
  for (int i = 0; i < NLA; ++i) {
    int r = min(i * 32 + (tid >> 3), rows_valid - 1);
    if (p.src_assign) r = a_row_of(p, tc.m_begin + r);
    soff_a[i] = static_cast<uint32_t>(r) * static_cast<uint32_t>(K) * 4u + static_cast<uint32_t>(chunk) * 16u;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
    soff_w[h] = static_cast<uint32_t>(min(wave * 16 + l16, N - 1 - n0)) * static_cast<uint32_t>(K) * 4u +
                static_cast<uint32_t>(kg + 4 * h) * 16u;
  const int tail_chunks = (K & (F32_BK - 1)) >> 2;
  auto past_end = [&](int kt, int c) { return kt >= KT || (tail_chunks != 0 && c >= tail_chunks) ? PAST_END : 0u; };
  f32x4_t va[NLA], vw[NMAT][2];
  auto load_a = [&](int kt) {
    if (kt >= KT - 1) {                           // uniform
#pragma unroll
      for (int i = 0; i < NLA; ++i) soff_a[i] |= past_end(kt, chunk);
    }
#pragma unroll
    for (int i = 0; i < NLA; ++i)
      va[i] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs.a, static_cast<int>(soff_a[i]), kt * ROWB, 0));
  };
  auto load_w = [&](int kt) {
    if (kt >= KT - 1) {
#pragma unroll
      for (int h = 0; h < 2; ++h) soff_w[h] |= past_end(kt, kg + 4 * h);
    }
#pragma unroll
    for (int m = 0; m < NMAT; ++m)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        vw[m][h] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(m ? rs.b1 : rs.b0, static_cast<int>(soff_w[h]), kt * ROWB, 0));
  };
  // plane row: four 16-byte chunks, chunk j = the row's 4-value chunks j and j + 4
  const int wr = (tid >> 3) * F32_PROW + (((chunk & 3) ^ swz64(tid >> 3)) << 4) + (chunk >> 2) * 8;
  auto split_a = [&](int buf) {
    unsigned char* to = lds + buf * STAGE + wr;
#pragma unroll
    for (int i = 0; i < NLA; ++i) {
      uint2 q[3];
      f32_split(va[i], q);
#pragma unroll
      for (int j = 0; j < 3; ++j) *reinterpret_cast<uint2*>(to + i * 32 * F32_PROW + j * F32_PLANE) = q[j];
    }
  };
  bf16x8_t wf[NMAT][3];
  auto split_w = [&]() {
#pragma unroll
    for (int m = 0; m < NMAT; ++m) {
      uint2 q0[3], q1[3];
      f32_split(vw[m][0], q0);
      f32_split(vw[m][1], q1);
#pragma unroll
      for (int j = 0; j < 3; ++j) wf[m][j] = __builtin_bit_cast(bf16x8_t, make_uint4(q0[j].x, q0[j].y, q1[j].x, q1[j].y));
    }
  };
  const int x_base = l16 * F32_PROW + ((kg ^ swz64(l16)) << 4);
  f32x4_t acc[NMAT][MI], rest[GATED ? 1 : MI][NMAT];
#pragma unroll
  for (int m = 0; m < NMAT; ++m)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      acc[m][mi] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      rest[GATED ? 0 : mi][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

  load_a(0);
  load_w(0);
  split_a(0);
  load_a(1);
  lds_barrier();
  auto k_loop = [&](auto miv_c) {
    constexpr int MIV = decltype(miv_c)::value;
    int buf = 0;
    for (int kt = 0; kt < KT; ++kt, buf ^= 1) {
      const unsigned char* s = lds + buf * STAGE + x_base;
      bf16x8_t x[2][3];
      auto read_x = [&](int mi) {
#pragma unroll
        for (int j = 0; j < 3; ++j) x[mi & 1][j] = *reinterpret_cast<const bf16x8_t*>(s + j * F32_PLANE + mi * 16 * F32_PROW);
      };
      read_x(0);
      split_w();
      load_w(kt + 1);
#pragma unroll
      for (int mi = 0; mi < MIV; ++mi) {
        if (mi + 1 < MIV) read_x(mi + 1);
        f32x4_t (&low)[NMAT] = rest[GATED ? 0 : mi];
        constexpr int WQ[7] = {2, 1, 2, 0, 1, 1, 0}, XQ[7] = {1, 2, 0, 2, 1, 0, 1};
#pragma unroll
        for (int t = 0; t < 7; ++t)
#pragma unroll
          for (int m = 0; m < NMAT; ++m)
            low[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[m][WQ[t]], x[mi & 1][XQ[t]], low[m], 0, 0, 0);
#pragma unroll
        for (int m = 0; m < NMAT; ++m)
          acc[m][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[m][0], x[mi & 1][0], acc[m][mi], 0, 0, 0);
        if constexpr (GATED) {
#pragma unroll
          for (int m = 0; m < NMAT; ++m) {
            acc[m][mi] += low[m];
            low[m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          }
        }
        if (mi == 0) {
          split_a(buf ^ 1);                       // (last read before the barrier of stage kt - 1)
          load_a(kt + 2);
        }
        asm volatile("" ::: "memory");            // one sub-tile's fragments ahead, not all of them
      }
      lds_barrier();
    }
  };
  switch ((rows_valid + 15) >> 4) {               // block-uniform
    case 1: k_loop(std::integral_constant<int, 1>{}); break;
    case 2: k_loop(std::integral_constant<int, 2>{}); break;
    case 3: k_loop(std::integral_constant<int, 3>{}); break;
    default: k_loop(std::integral_constant<int, 4>{}); break;
  }
  if constexpr (!GATED) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) acc[0][mi] += rest[mi][0];
  }
  bool finite = true;
#pragma unroll
  for (int m = 0; m < NMAT; ++m)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int u = 0; u < 4; ++u) finite = finite && __builtin_isfinite(acc[m][mi][u]);
  if (!__syncthreads_and(finite)) return false;
  f32_store<GATED, MI>(acc, p, n0, tc.m_begin, tc.m_end, F32_UNSCALE);
  return true;
}

// SPLIT: a launch of 64-row tiles, which takes the split path where a tile has more than 32 rows.
template <bool GATED, bool SPLIT>
__global__ __launch_bounds__(F32_NW * MOE_WAVE, 3) void ffn_f32_kernel(GemmArgs p) {
  extern __shared__ __align__(1024) unsigned char lds[];
  TileCoord tc;
  if (!decode_tile(p, tc)) return;
  if constexpr (!SPLIT) {
    f32_exact_rows<GATED>(p, tc, lds, tc.m_begin, tc.m_end);
  } else {
    if (tc.m_end - tc.m_begin > F32_EXACT_ROWS && f32_split_tile<GATED>(p, tc, lds)) return;
    for (int m = tc.m_begin; m < tc.m_end; m += F32_EXACT_ROWS) {
      lds_barrier();                              // (the rows before, or the split path, have left the LDS)
      f32_exact_rows<GATED>(p, tc, lds, m, min(m + F32_EXACT_ROWS, tc.m_end));
    }
  }
}

// --------------------------------------------------------------------------------------------
// Very wide layers (a tile's operand spans 2 GiB or more, see tile_fits): 64 x 64 output tile, K step 16,
// 4 x 4 outputs per thread, fp32 FMA, 64-bit addresses throughout.  Bound by the vector pipe (50 TFLOP/s
// where there are tiles enough); no model is this wide, the kernel keeps such calls right.
// --------------------------------------------------------------------------------------------
constexpr int WIDE_T = 64;
__device__ __forceinline__ float ld_elem(const float* p) { return *p; }
__device__ __forceinline__ float ld_elem(const bf16_t* p) { return bf16_to_f32(*p); }
__device__ __forceinline__ void st_elem(float* p, float v) { *p = v; }
__device__ __forceinline__ void st_elem(bf16_t* p, float v) { *p = f32_to_bf16(v); }

template <typename T, bool GATED>
__global__ __launch_bounds__(256) void ffn_wide_kernel(GemmArgs p) {
  constexpr int TK = 16, NMAT = GATED ? 2 : 1;
  __shared__ float As[TK][WIDE_T + 4];
  __shared__ float Bs[NMAT][TK][WIDE_T + 4];
  TileCoord tc;
  if (!decode_tile(p, tc)) return;
  const int64_t K = p.K;
  const int N = p.N, n0 = tc.n0;
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;         // thread's 4 columns / 4 rows
  const int lr = tid >> 2, lk = (tid & 3) * 4;    // loader: row 0..63, k offset 0,4,8,12
  const T* a = static_cast<const T*>(p.a) + a_row_of(p, min(tc.m_begin + lr, tc.m_end - 1)) * K;
  const int64_t b_off = (static_cast<int64_t>(tc.e) * N + min(n0 + lr, N - 1)) * K;
  const T* b[NMAT];
  b[0] = static_cast<const T*>(p.b0) + b_off;
  if constexpr (GATED) b[1] = static_cast<const T*>(p.b1) + b_off;
  float acc[NMAT][4][4] = {};
  for (int64_t k0 = 0; k0 < K; k0 += TK) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t kk = k0 + lk + q;
      As[lk + q][lr] = kk < K ? ld_elem(a + kk) : 0.f;
#pragma unroll
      for (int m = 0; m < NMAT; ++m) Bs[m][lk + q][lr] = kk < K ? ld_elem(b[m] + kk) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < TK; ++kk)
#pragma unroll
      for (int m = 0; m < NMAT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[m][i][j] = fmaf(As[kk][ty * 4 + i], Bs[m][kk][tx * 4 + j], acc[m][i][j]);
    __syncthreads();
  }
  T* out = static_cast<T*>(p.out);
  const int32_t* out_map = GATED ? nullptr : p.out_map;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int gr = tc.m_begin + ty * 4 + i;
    if (gr >= tc.m_end) continue;
    float scale = 1.f;
    if (out_map) {
      gr = min(max(out_map[gr], 0), p.out_rows - 1);
      scale = p.out_scale[gr];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = n0 + tx * 4 + j;
      if (c >= N) continue;
      const float v = acc[0][i][j];
      st_elem(out + static_cast<int64_t>(gr) * N + c,
              GATED ? silu_mul<true>(v, acc[NMAT - 1][i][j]) : out_map ? v * scale : v);
    }
  }
}

// Upper bound on the number of m-tiles that needs no knowledge of the counts: an expert with c rows
// has ceil(c / bm) <= c / bm + 1 tiles, and at most min(E, A) experts have any.
static int64_t max_m_tiles(int64_t A, int E, int bm) { return A / bm + (E < A ? E : A); }

// `split`: the launch may use the workspace for split tiles if the caller brought one.  Only
// GEMMs with a long reduction do: a part must be worth the exchange (one store of 64 to 320 KiB of
// accumulators per part, the summing launch), and a tile of fewer than 96 stages is too short for that (measured:
// the up-projections of the four model shapes gain nothing, their down-projections up to 27 %).
constexpr int SPLIT_MIN_K = 96 * BK_ELEMS;

// One grouped GEMM.  main_kernel: void (*)(GemmArgs); the grid is an upper bound of the tile count
// (surplus blocks exit at once), plus a round of blocks for the parts when tiles may be split; the
// summing kernel (one block per possible split tile) follows on the same stream.
static int launch_grouped_gemm(GemmArgs a, int bm, int64_t A, int threads, int lds_bytes,
                               void (*main_kernel)(GemmArgs), LdsOnce& once_main,
                               void (*sum_kernel)(GemmArgs), LdsOnce& once_sum, hipStream_t st) {
  if (ensure_dynamic_lds(once_main, reinterpret_cast<const void*>(main_kernel), lds_bytes) != MOE_OK)
    return MOE_ERR_HIP;
  a.bm = bm;
  a.split_phase = 0;
  if (!sum_kernel) a.split_ws = nullptr;
  int64_t grid = max_m_tiles(A, a.E, bm) * a.n_tiles;
  if (grid == 0) return MOE_OK;
  grid = (grid + 7) / 8 * 8;
  const int cu8 = (a.n_cu > 0 ? a.n_cu : 256) / 8 * 8;
  if (sum_kernel || a.tail_split) grid += cu8;
  if (grid > 0x7FFFFFFF) return MOE_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(main_kernel, dim3(static_cast<unsigned>(grid)), dim3(threads), lds_bytes, st, a);
  int rc = launch_status();
  if (sum_kernel && rc == MOE_OK) {
    if (ensure_dynamic_lds(once_sum, reinterpret_cast<const void*>(sum_kernel), lds_bytes) != MOE_OK)
      return MOE_ERR_HIP;
    a.split_phase = 1;
    hipLaunchKernelGGL(sum_kernel, dim3(static_cast<unsigned>(cu8)), dim3(threads), lds_bytes, st, a);
    rc = launch_status();
  }
  return rc;
}

// Shapes the RAGGED kernels take (they are not cut along K: a workspace is ignored).
static bool ragged(const GemmArgs& a) { return a.K % BK_ELEMS != 0 || a.N % BK_ELEMS != 0; }

// Most rows of a bf16 tile, by the mean rows per expert.  Below 128 rows most experts are one tile under
// either limit; what the limit changes is a hot expert of a skewed batch, whose few high tiles would be the
// launch's longest.  (Measured, whole layer, limit 320 against the one below: skewed 64-expert layer at
// 512 / 680 tokens, 48 and 64 rows per expert, 270 / 311 -> 244 / 267 us; at 1024 tokens, 96 rows,
// 342 -> 317 us with 192; unskewed layers within 1 %.  With 192 up to 192 rows per expert the
// 128-expert layer at 2500 tokens is 4 % slower.)
static int most_tile_rows(int64_t mean_rows) { return mean_rows < 96 ? 128 : mean_rows < 128 ? 192 : EVEN_BM; }

// The MFMA kernels address a tile's rows of an operand by 32-bit byte offsets from its first row, below the
// 2 GiB that a buffer resource admits (requests beyond it come back as zeros: see PAST_END).  True if
// `rows` rows of the GEMM's reduction stay inside.
static bool tile_fits(const GemmArgs& a, int rows, int elem) {
  return static_cast<int64_t>(rows) * a.K * elem < (int64_t(1) << 31);
}

template <typename T, bool GATED>
static int launch_wide(GemmArgs a, int64_t A, hipStream_t st) {
  static LdsOnce once[2];
  a.bn = WIDE_T;
  a.n_tiles = (a.N + WIDE_T - 1) / WIDE_T;
  return launch_grouped_gemm(a, WIDE_T, A, 256, 0, ffn_wide_kernel<T, GATED>, once[0], nullptr, once[1], st);
}

// Mean rows per expert from which most experts are two tiles or more.
constexpr int FEW_BUFFERS_ROWS = 384;

template <bool GATED, bool WNT>
static int launch_bf16(GemmArgs a, int64_t A, bool row_split, hipStream_t st) {
  static LdsOnce once[2], once_ragged, once_sum;
  const int bm = most_tile_rows(A / a.E);
  if (!tile_fits(a, bm > BROWS ? bm : BROWS, 2)) return launch_wide<bf16_t, GATED>(a, A, st);
  // Two tiles of 192 to 256 rows that share their weight rows gain from a third buffer in the up-projection
  // unless the row pitch is a power of two, which puts a tile's 256 rows on few memory channels.
  // (Measured, three against two buffers, 16 experts of 400 / 460 rows, F = 6400, up-projection: d = 3072
  // 8 / 3 % faster, 5120 8 / 7 %, 6144 9 / 5 %, 4608 and 7168 within 3 % either way, 4096 3 % slower, 2048
  // 2 % faster / 3 % slower; below 384 rows faster at every d, 2 to 11 %.)
  a.few_buffers = GATED && A / a.E >= FEW_BUFFERS_ROWS && (a.K & (a.K - 1)) == 0;
  GemmArgs b = a;
  b.tail_split = row_split ? 1 : 0;
  if (ragged(a))
    return launch_grouped_gemm(b, bm, A, 512, FFN_LDS,
                               ffn_bf16_kernel<GATED, false, true, true>, once_ragged, nullptr, once_sum, st);
  if (a.split_ws && a.K >= SPLIT_MIN_K)
    return launch_grouped_gemm(a, bm, A, 512, FFN_LDS,
                               ffn_bf16_kernel<GATED, true, WNT, false>, once[1],
                               ffn_bf16_sum_parts_kernel<GATED, WNT>, once_sum, st);
  return launch_grouped_gemm(b, bm, A, 512, FFN_LDS,
                             ffn_bf16_kernel<GATED, false, WNT, false>, once[0], nullptr, once_sum, st);
}

// 64-row tiles, which take the split path, from F32_SPLIT_ROWS rows per expert on, if there are more than 5/4 for every
// CU; 32-row tiles, on the fp32 instruction, below.  (Measured, 32-row against 64-row tiles, us.  Rows per expert, both
// GEMMs: d = 1024, E = 40, F = 2048, 26 rows 230 / 242, 32 231 / 232, 36 259 / 230, 44 285 / 265; d = F = 768, E = 64, 36 rows
// 123 / 102, 64 156 / 155, 200 396 / 370.  Tiles, with few of which a tile's stages are a serial chain, longer with the cutting,
// each GEMM: 256 tiles 58 / 66 and 153 / 170, 304 66 / 72, 320 58 / 66 and 73 / 60; 340 85 / 80, 352 78 / 68, 384 73 / 68 and
// 198 / 185.)
constexpr int F32_SPLIT_ROWS = 36;
template <bool GATED>
static int launch_f32(GemmArgs a, int64_t A, hipStream_t st) {
  static LdsOnce once[2], once_sum;
  if (!tile_fits(a, F32_BN, 4)) return launch_wide<float, GATED>(a, A, st);
  a.bn = F32_BN;
  a.n_tiles = (a.N + F32_BN - 1) / F32_BN;
  const int64_t tiles = (A + F32_BM - 1) / F32_BM * a.n_tiles;
  if (A / a.E >= F32_SPLIT_ROWS && 4 * tiles > 5 * static_cast<int64_t>(a.n_cu > 0 ? a.n_cu : 256))
    return launch_grouped_gemm(a, F32_BM, A, F32_NW * MOE_WAVE, ffn_f32_lds_bytes(GATED),
                               ffn_f32_kernel<GATED, true>, once[0], nullptr, once_sum, st);
  return launch_grouped_gemm(a, F32_EXACT_ROWS, A, F32_NW * MOE_WAVE, ffn_f32_lds_bytes(GATED),
                             ffn_f32_kernel<GATED, false>, once[1], nullptr, once_sum, st);
}

// Mean rows per expert below which the kernels are built with the per-tile choice of the
// non-temporal hint for weight rows (experts of at most two tiles are then the rule).
constexpr int WGT_NT_ROWS = 2 * EVEN_BM;

// Both GEMMs (or one of them) on the MFMA path: one launch each on the caller's stream.
static int mfma_ffn(GemmArgs g1, GemmArgs g2, bool up, bool down, int64_t A, bool row_split,
                    hipStream_t st) {
  int rc = MOE_OK;
  if (A / g1.E >= WGT_NT_ROWS) {
    if (up && (rc = launch_bf16<true, false>(g1, A, row_split, st)) != MOE_OK) return rc;
    if (down) rc = launch_bf16<false, false>(g2, A, row_split, st);
  } else {
    if (up && (rc = launch_bf16<true, true>(g1, A, row_split, st)) != MOE_OK) return rc;
    if (down) rc = launch_bf16<false, true>(g2, A, row_split, st);
  }
  return rc;
}

// parts: bit 0 = gated up-projection (h), bit 1 = down-projection (y_perm)
// x_perm [T*k, d] with src_assign == nullptr, or x [T, d] with the src_assign map of the dispatch
// combine_w != nullptr (k = 1 layers only): y_perm is y [T, d]; row r of the down-projection is
// stored to y[src_assign[r]] times combine_w[src_assign[r]]
static int grouped_ffn_impl(const moe_shape_t* shape, const void* x_perm, const int32_t* src_assign,
                            const int32_t* offsets, const void* w1, const void* w3, const void* w2,
                            void* h, void* y_perm, int parts, void* hip_stream,
                            void* split_ws = nullptr, const float* combine_w = nullptr,
                            bool row_split = true) {
  int rc = check_shape(shape);
  if (rc != MOE_OK) return rc;
  if (shape->T == 0) return MOE_OK;
  if (!x_perm || !offsets || !w1 || !w3 || !w2 || !h || !y_perm) return MOE_ERR_INVALID_ARG;
  // gathered rows are addressed with a 32-bit byte offset from the start of x
  if (src_assign && static_cast<int64_t>(shape->T) * shape->d * elem_bytes(shape->dtype) >=
                        (int64_t(1) << 31))
    return MOE_ERR_UNSUPPORTED;
  if (!aligned16(x_perm) || !aligned16(w1) || !aligned16(w3) || !aligned16(w2) || !aligned16(h) ||
      !aligned16(y_perm))
    return MOE_ERR_INVALID_ARG;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int64_t A = static_cast<int64_t>(shape->T) * shape->k;
  const int d = shape->d, F = shape->F, E = shape->E;
  const int n_cu = device_cu_count();
  GemmArgs g1{x_perm, w1, w3, h, offsets, E, d, F, 0, 0, static_cast<int>(A), EVEN_BM,
              src_assign, shape->k, src_assign ? shape->T : static_cast<int>(A), n_cu,
              static_cast<float*>(split_ws), 0, nullptr, nullptr, 0};
  GemmArgs g2{h, w2, nullptr, y_perm, offsets, E, F, d, 0, 0, static_cast<int>(A), EVEN_BM,
              nullptr, 1, static_cast<int>(A), n_cu, static_cast<float*>(split_ws), 0,
              combine_w ? src_assign : nullptr, combine_w, shape->T};
  const bool up = parts & 1, down = parts & 2;
  if (shape->dtype == MOE_BF16) {
    g1.bn = 128;
    g2.bn = 256;
    g1.n_tiles = (F + g1.bn - 1) / g1.bn;
    g2.n_tiles = (d + g2.bn - 1) / g2.bn;
    return mfma_ffn(g1, g2, up, down, A, row_split, st);
  }
  if (up) {
    rc = launch_f32<true>(g1, A, st);
    if (rc != MOE_OK) return rc;
  }
  if (down) rc = launch_f32<false>(g2, A, st);
  return rc;
}

}  // namespace moe

extern "C" int moe_grouped_ffn(const moe_shape_t* shape, const void* x_perm, const int32_t* offsets,
                               const void* w1, const void* w3, const void* w2, void* h, void* y_perm,
                               void* hip_stream) {
  return moe::grouped_ffn_impl(shape, x_perm, nullptr, offsets, w1, w3, w2, h, y_perm, 3,
                               hip_stream);
}

// Bytes of the split-tile workspace on the current device: one fp32 partial tile per compute unit.
static size_t ffn_split_workspace_bytes() {
  const int n_cu = moe::device_cu_count();
  return static_cast<size_t>(n_cu > 0 ? n_cu : 256) * moe::SPLIT_SLOT_FLOATS * sizeof(float);
}

extern "C" int moe_ffn_workspace_bytes(const moe_shape_t* shape, size_t* out_bytes) {
  if (!out_bytes) return MOE_ERR_INVALID_ARG;
  const int rc = moe::check_shape(shape);
  if (rc != MOE_OK) return rc;
  *out_bytes = ffn_split_workspace_bytes();
  return MOE_OK;
}

extern "C" int moe_grouped_ffn_ws(const moe_shape_t* shape, const void* x, const int32_t* src_assign,
                                  const int32_t* offsets, const void* w1, const void* w3,
                                  const void* w2, void* h, void* y_perm, int parts, void* workspace,
                                  size_t workspace_bytes, void* hip_stream) {
  const bool whole_tiles = (parts & 4) != 0;
  parts &= ~4;
  if (parts < 1 || parts > 3) return MOE_ERR_INVALID_ARG;
  if (workspace) {
    if (!moe::aligned16(workspace)) return MOE_ERR_INVALID_ARG;
    if (workspace_bytes < ffn_split_workspace_bytes()) return MOE_ERR_WORKSPACE;
  }
  return moe::grouped_ffn_impl(shape, x, src_assign, offsets, w1, w3, w2, h, y_perm, parts,
                               hip_stream, workspace, nullptr, !whole_tiles);
}

extern "C" int moe_grouped_ffn_gather(const moe_shape_t* shape, const void* x,
                                      const int32_t* src_assign, const int32_t* offsets,
                                      const void* w1, const void* w3, const void* w2, void* h,
                                      void* y_perm, void* hip_stream) {
  if (!src_assign) return MOE_ERR_INVALID_ARG;
  return moe::grouped_ffn_impl(shape, x, src_assign, offsets, w1, w3, w2, h, y_perm, 3, hip_stream);
}

extern "C" int moe_grouped_ffn_combine_k1(const moe_shape_t* shape, const void* x,
                                          const int32_t* src_assign, const int32_t* offsets,
                                          const void* w1, const void* w3, const void* w2,
                                          const float* topk_w, void* h, void* y, void* hip_stream) {
  if (!shape) return MOE_ERR_INVALID_ARG;
  if (shape->k != 1) return MOE_ERR_UNSUPPORTED;
  if (!src_assign || !topk_w) return MOE_ERR_INVALID_ARG;
  return moe::grouped_ffn_impl(shape, x, src_assign, offsets, w1, w3, w2, h, y, 3, hip_stream, nullptr,
                               topk_w);
}

extern "C" int moe_grouped_ffn_gather_part(const moe_shape_t* shape, const void* x,
                                           const int32_t* src_assign, const int32_t* offsets,
                                           const void* w1, const void* w3, const void* w2, void* h,
                                           void* y_perm, int part, void* hip_stream) {
  if (part != 1 && part != 2) return MOE_ERR_INVALID_ARG;
  if (!src_assign) return MOE_ERR_INVALID_ARG;
  return moe::grouped_ffn_impl(shape, x, src_assign, offsets, w1, w3, w2, h, y_perm, part,
                               hip_stream);
}

extern "C" int moe_grouped_ffn_part(const moe_shape_t* shape, const void* x_perm,
                                    const int32_t* offsets, const void* w1, const void* w3,
                                    const void* w2, void* h, void* y_perm, int part,
                                    void* hip_stream) {
  if (part != 1 && part != 2) return MOE_ERR_INVALID_ARG;
  return moe::grouped_ffn_impl(shape, x_perm, nullptr, offsets, w1, w3, w2, h, y_perm, part,
                               hip_stream);
}
