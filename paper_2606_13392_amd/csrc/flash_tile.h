// Query-tile-outer softmax attention on gfx950 (FlashAttention-2 order),
// shared by the dense baseline and by the prefill Main Branch on rows whose
// selection covers much of their causal context.
//
// A CTA owns one KV group and a tile of consecutive query rows of one sequence
// whose G heads share the group's K and V; each of its waves holds 32 (query
// row, head) rows.  Key sub-blocks of 64 go through a double-buffered LDS ring
// one sub-block ahead (bf16: DMA, global_load_lds; E4M3: through registers,
// widened to bf16 on the way), rows stored with a bank-conflict-free segment
// permutation; per sub-block each wave computes S^T = K Q^T and
// O^T += V^T P^T with MFMA 32x32x16, the V^T operand read down V's columns
// with transposing LDS reads.  The O MFMAs of one sub-block are interleaved by
// hand with the online softmax of the next (running max and sum per row in
// registers, raw hardware exp2).
//
// SPARSE: the tile's block ids become one word per (wave, key block), bit j
// set when the wave's row j selected the block; the CTA walks the blocks some
// row selected, and a row that did not select the block takes part with weight
// zero (its exponent offset is -inf: two instructions per row and sub-block,
// none per score).  (Skipping a block in the waves none of whose rows selected
// it needs the score, softmax and value phases apart from one another: the
// merged control flow spilled 65 - 130 registers.)  No partial leaves the CTA.
// Weight zero hides finite keys and values only; a NaN or infinity in a block
// would reach the rows that did not select it, always as a NaN in their sum or
// output.  A tile that ends with one walks its blocks again, one at a time,
// with a selection per row in place of the zero weights (the same results to
// the bit where the inputs are finite).
//
// CTAs are ordered group-fastest: consecutive CTAs go to different XCDs, so
// each XCD's L2 holds the K / V of its own groups, and every group's longest
// tiles start first.  The dense call orders them tile-fastest where a
// sequence's K and V outgrow the last-level cache (Grid, kCacheBytes).
#pragma once

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "msa_common.h"
#include "msa_profile.h"

namespace {

using namespace msa;

namespace flash {

constexpr int kDim = 128;                // head dimension
constexpr int kSub = 64;                 // keys per streamed sub-block
constexpr float kLog2E = 1.4426950408889634f;
constexpr float kLn_2 = 0.6931471805599453f;
constexpr int kAhead = 3;                // LDS operand reads issued this many MFMA slots ahead
constexpr int kMaxBlocks = 256;          // key blocks a sparse tile may reach back over

// Key sub-blocks in LDS, row-major, 16-byte segments permuted per row (an XOR
// with a row-dependent mask) so that every read pattern is free of bank
// conflicts whether the LDS serves 16 or 32 lanes of a wave per cycle:
//   K (16 bytes per lane: 32 consecutive rows x the two segments of a k-step)
//     segment s of row r at s ^ (2 (r & 7) + ((r >> 3) & 1));
//   V (ds_read_tr16_b64: 4 consecutive rows x 4 adjacent segments per 32
//     lanes) segment s of row r at s ^ 4 (r & 3).
struct Ring {
  uint16_t k[2][kSub * kDim];
  uint16_t v[2][kSub * kDim];
};
__device__ __forceinline__ int k_seg(int r, int s) { return s ^ (((r & 7) << 1) | ((r >> 3) & 1)); }
__device__ __forceinline__ int v_seg(int r, int s) { return s ^ ((r & 3) << 2); }

// The blocks a sparse tile visits.
template <int WAVES, int SUB>
struct Visits {
  uint32_t rows[WAVES][kMaxBlocks];      // bit j: the wave's query row j selected the block
  uint32_t at[kMaxBlocks * SUB];         // per visited sub-block: its first key row / 64 (paged: in the pool)
  uint16_t sub[kMaxBlocks * SUB];        // ... and its index in the sequence
  int32_t n;
  int32_t redo;                          // some row's result is not finite
};
struct NoVisits {};

// lsum + lo + hi of a packed bf16 pair (v_dot2c_f32_bf16 against (1, 1)):
// the row sum is taken over the same rounded weights that multiply V.
__device__ __forceinline__ float add_bf16_pair(float lsum, uint32_t pair) {
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2v;
  const bf16x2v ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, pair), ones, lsum, false);
}
__device__ __forceinline__ float xor32f(float x) {
  return __builtin_bit_cast(float, xor_lane_u32<32>(__builtin_bit_cast(uint32_t, x)));
}
__device__ __forceinline__ uint2 lds_tr4(const uint16_t* p) {
  typedef __attribute__((__vector_size__(4 * sizeof(short)))) short v4i16;
  const v4i16 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) v4i16*)(v4i16*)(const_cast<uint16_t*>(p)));
  return __builtin_bit_cast(uint2, x);
}
// global_load_lds: lane l's 16 bytes land at dst + 16 l (dst wave-uniform).
__device__ __forceinline__ void dma16(const void* src, uint16_t* dst) {
  __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

// Per-lane byte offsets of one sub-block's copies (global side, relative to
// its first key row) and of the MFMA operand reads (LDS side, relative to a
// ring buffer), fixed for the whole kernel.
template <int NDMA>
struct LaneOffsets {
  uint32_t kg[NDMA], vg[NDMA];           // DMA sources: row * stride + 16-byte segment
  uint32_t ks[kDim / 16];                // K operand, k-step st (rows 32i add 8 KiB)
  uint32_t vs[kDim / 32];                // V^T operand, dim tile td (row offsets are immediates)
};

// Tiles of the grid (x H_kv CTAs, group fastest), the last tile of the last
// sequence first.  Sequence s owns tiles from q_offsets[s] / qt + s on, at
// least as many as it needs, so at most one tile per sequence is empty.  (The
// dispatcher deals CTAs to shader engines in turn, so empty CTAs between the
// others unbalance it: the longest tiles first over all sequences, with empty
// slots for the shorter ones, took 677 us instead of 486 for 1427 + 4846
// rows; and a sequence at a time keeps its K and V in L2.)  A single sequence
// has no tiles past max_rows.
struct Grid {
  int32_t tiles;
  bool tile_fast;                        // dense: all tiles of a group, then the next group's
};
// A dense sequence with more K and V than the last-level cache (256 MiB) runs
// one group at a time: all CTAs stream the same K and V, which then come from
// that cache for all XCDs but the first to ask.  Group-fastest every XCD is the
// first to ask for its own group's.  A prompt, whose tiles differ in length,
// does so only with many tiles per group (kManyTiles): the last group's longest
// tile starts late.  Group-fastest against tile-fastest on MI355X, heads on
// groups: 64 on 8 (4 KiB per key), prompts of 32768 keys 15.7 / 16.0 ms, 49152
// 35.3 / 35.5, 65536 63.1 / 62.7, 131072 257 / 249; 8192 rows on 1M keys 258 /
// 246; 12 sequences of 3000 keys 1.68 / 1.81.  Prompts, 16 on 16, 32768 keys
// (128 tiles) 4.3 / 5.1, 98304 (384) 38.0 / 37.9; 64 on 16, 32768 (512) 16.4 /
// 16.7, 65536 (1024) 67.4 / 65.4.  8192 rows on 64K keys, 32 on 32: 9.3 / 9.1.
constexpr int64_t kCacheBytes = int64_t(1) << 28;
constexpr int64_t kManyTiles = 1024;
inline bool tile_fast(const msa_seqs* seqs, int H_kv, int qt) {
  const int64_t keys = seqs->max_kv_len, rows = seqs->max_q_rows;
  return keys * H_kv * (2 * kDim * 2) >= kCacheBytes && (2 * rows <= keys || rows >= kManyTiles * qt);
}
inline Grid plan_grid(const msa_seqs* seqs, int qt, int64_t max_rows, int64_t* tiles) {
  *tiles = seqs->num_seqs == 1 ? (std::min<int64_t>(seqs->max_q_rows, max_rows) + qt - 1) / qt
                               : seqs->total_q_rows / qt + seqs->num_seqs;
  return Grid{static_cast<int32_t>(std::min<int64_t>(*tiles, 0x7FFFFFFF)), false};
}
// Sequence and tile of grid tile `u` (wave-uniform).
__device__ __forceinline__ void locate_tile(const msa_seqs& sq, const Grid& gr, int u, int qt, int* seq, int* tile) {
  const int x = gr.tiles - 1 - u;
  int lo = 0, n = sq.num_seqs;           // the answer lies in [lo, lo + n)
  while (n > 1) {
    const int stride = (n + kWave - 1) / kWave;
    const int idx = lo + lane_id() * stride;
    const bool ok = idx < lo + n && sq.q_offsets[idx] / qt + idx <= x;
    const uint64_t mask = __ballot(ok);  // a prefix of the lanes: the starts increase
    const int j = 63 - __clzll(static_cast<long long>(mask | 1ull));
    const int lo_new = lo + j * stride;
    n = min(stride, lo + n - lo_new);
    lo = lo_new;
  }
  *seq = lo;
  *tile = x - (sq.q_offsets[lo] / qt + lo);
}

// The kernel masks and takes maxima of raw scores, so its scale is positive: a
// negative one flips the signs of Q (S and the scale change sign together,
// exactly), and a zero one becomes the smallest normal number (no exponent of
// scores below 2^100 then differs from 0 by more than 2^-26).
struct LogitScale {
  float log2;                            // > 0 (NaN stays)
  uint32_t q_flip;                       // XORed into bf16 pairs of Q
};
inline LogitScale logit_scale(float scale_log2) {
  const float a = std::fabs(scale_log2);
  return LogitScale{a < FLT_MIN ? FLT_MIN : a, scale_log2 < 0.f ? 0x80008000u : 0u};
}

// T: element type of q, k and v (uint16_t = bf16 bits, uint8_t = e4m3 bits;
// o_scale multiplies O).  SPARSE: block ids of BK keys per (row, group), rows
// at positions below p_cut (at most kMaxBlocks * BK); else every causal key.
//
// Per iteration b (one barrier): the copies of K_{b+2} and V_{b+1} are issued,
// S^T_{b+1} = K_{b+1} Q^T and O^T += V_b^T P_b^T are issued on the MFMA pipe,
// and the softmax of S_{b+1} runs on the VALU while the O MFMAs drain.
template <typename T, int BK, bool SPARSE, bool PAGED, int WAVES>
__global__ __launch_bounds__(WAVES* kWave, 2) void flash_tile_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const int32_t* __restrict__ block_ids, msa_seqs sq, Grid gr, int H_q, int H_kv, int topk, int p_cut,
    float scale_log2, uint32_t q_flip, float o_scale, uint16_t* __restrict__ o, float* __restrict__ lse) {
  constexpr int SUB = BK / kSub;           // 64-key sub-blocks per block
  constexpr int kThreads = WAVES * kWave;
  constexpr int MT = kSub / 32;            // 32-key tiles of S^T
  constexpr int KS = kDim / 16;            // k-steps of S^T = K Q^T
  constexpr bool kDma = sizeof(T) == 2;
  constexpr int NDMA = kSub / 4 / WAVES;   // DMA instructions per wave per sub-block and tensor
  constexpr int NRAW = kSub * kDim / 16 / kThreads;   // E4M3: 16-byte pieces per thread and tensor
  __shared__ __align__(16) Ring ring;
  __shared__ std::conditional_t<SPARSE, Visits<WAVES, SUB>, NoVisits> vis;
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  const int n = lane & 31, h = lane >> 5;
  const int G = H_q / H_kv;
  const int qpw = 32 / G;                  // query rows per wave
  const int qt = WAVES * qpw;              // query rows per CTA
  const int jq = n / G, hh = n % G;
  const bool by_tile = !SPARSE && gr.tile_fast;
  const unsigned inner = by_tile ? static_cast<unsigned>(gr.tiles) : static_cast<unsigned>(H_kv);
  const int fast = static_cast<int>(blockIdx.x % inner), slow = static_cast<int>(blockIdx.x / inner);
  const int r = by_tile ? slow : fast;
  int s, tile;
  locate_tile(sq, gr, by_tile ? fast : slow, qt, &s, &tile);
  const SeqGeom g = seq_geom(sq, s);
  const int t0 = tile * qt;
  const int base_p = g.kv_len - g.q_rows;  // position of the sequence's first query row
  int t_end = min(t0 + qt, g.q_rows);
  t_end = static_cast<int>(min(static_cast<int64_t>(t_end), sq.total_q_rows - g.q_begin));
  if constexpr (SPARSE) t_end = min(t_end, p_cut - base_p);
  if (t_end <= t0) return;                                // uniform over the CTA
  const int p_last = base_p + t_end - 1;
  if (!SPARSE && p_last < 0) return;
  const int t = t0 + wave * qpw + jq;                     // this lane's query row in the sequence
  const bool valid = n < qpw * G && t < t_end;
  const int p = valid ? base_p + t : -1;
  // sub-blocks below nfree are visible to every row of the wave and need no
  // causal mask (a wave without rows never looks)
  const int nfree = (base_p + min(t0 + wave * qpw, t_end - 1) + 1) / kSub;
  const int64_t head_row = (static_cast<int64_t>(g.q_begin) + (valid ? t : t0)) * H_q + static_cast<int64_t>(r) * G + hh;

  Raw<T> rq[KS];
  {
    const T* qrow = q + head_row * kDim + 8 * h;
#pragma unroll
    for (int st = 0; st < KS; ++st) rq[st] = valid ? load_raw(qrow + 16 * st) : Raw<T>{};
  }

  int nvisit = p_last / kSub + 1;                         // sub-blocks to visit
  if constexpr (SPARSE) {
    const int nb = p_last < 0 ? 0 : p_last / BK + 1;      // <= kMaxBlocks: p_last < p_cut
    for (int i = threadIdx.x; i < WAVES * kMaxBlocks; i += kThreads) vis.rows[i / kMaxBlocks][i % kMaxBlocks] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < (t_end - t0) * topk; i += kThreads) {
      const int j = i / topk;                             // row in the tile
      const int pj = base_p + t0 + j;
      const int b = block_ids[((static_cast<int64_t>(g.q_begin) + t0 + j) * H_kv + r) * topk + i % topk];
      if (pj >= 0 && b >= 0 && b <= pj / BK) atomicOr(&vis.rows[j / qpw][b], 1u << (j % qpw));
    }
    __syncthreads();
    if (wave == 0) {
      const KeyBlocks kbk = key_blocks(sq, g, s, BK);
      int cnt = 0;
      bool tail = false;                                  // the last block's second half lies past p_last
      for (int b0 = 0; b0 < nb; b0 += kWave) {
        const int b = b0 + lane;
        uint32_t any = 0;
        if (b < nb)
          for (int w = 0; w < WAVES; ++w) any |= vis.rows[w][b];
        const uint64_t m = __ballot(any != 0);
        if (any != 0) {
          const int pos = cnt + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                                          __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0));
          const uint32_t at = PAGED ? static_cast<uint32_t>(kbk.template row_as<PAGED>(b) / kSub)
                                    : static_cast<uint32_t>(b * SUB);
#pragma unroll
          for (int e = 0; e < SUB; ++e) {
            vis.at[pos * SUB + e] = at + e;
            vis.sub[pos * SUB + e] = static_cast<uint16_t>(b * SUB + e);
          }
        }
        if (SUB == 2) tail = tail || __ballot(any != 0 && (b * SUB + 1) * kSub > p_last) != 0;
        cnt += __popcll(m);
      }
      if (lane == 0) {
        vis.n = cnt * SUB - (tail ? 1 : 0);
        vis.redo = 0;
      }
    }
    __syncthreads();
    nvisit = vis.n;
  }

  const int64_t stride = static_cast<int64_t>(H_kv) * kDim;
  const int64_t key_base = PAGED ? 0 : g.kv_start;
  const char* kb = reinterpret_cast<const char*>(k + key_base * stride + static_cast<int64_t>(r) * kDim);
  const char* vb = reinterpret_cast<const char*>(v + key_base * stride + static_cast<int64_t>(r) * kDim);
  const uint32_t stride_b = static_cast<uint32_t>(stride * sizeof(T));

  LaneOffsets<NDMA> lo;
  {
    const int gq = lane >> 4, jj = lane & 15;
#pragma unroll
    for (int c = 0; c < NDMA; ++c) {
      const int ra = 4 * (c * WAVES + wave) + gq;
      lo.kg[c] = ra * stride_b + 16 * k_seg(ra, jj);        // the permutations are involutions
      lo.vg[c] = ra * stride_b + 16 * v_seg(ra, jj);
    }
#pragma unroll
    for (int st = 0; st < KS; ++st) lo.ks[st] = 2 * (n * kDim + 8 * k_seg(n, 2 * st + h));
    // V^T operand: in each 16-lane group, lane j addresses row k0 + j/4, dims
    // n0 + 4(j%4) .. +3 of V and receives rows k0 .. k0+3 of dim n0 + j
    // (ds_read_tr16_b64); row r_l = 4h + j/4 within each 16-key k-step (rows
    // 16u + r_l and + 8 share the permutation)
    const int rl = 4 * h + (jj >> 2);
#pragma unroll
    for (int td = 0; td < kDim / 32; ++td) {
      const int col = 32 * td + 16 * (gq & 1) + 4 * (jj & 3);
      lo.vs[td] = 2 * (rl * kDim + 8 * v_seg(rl, col >> 3) + (col & 7));
    }
  }
  // One sub-block (K or V) into LDS by DMA: each wave instruction fills 4 rows
  // (1 KiB); lane l takes row 4 piece + l / 16 and the logical segment that
  // the row's permutation stores at physical segment l % 16.  In a sub-block
  // running past kv_len the missing rows re-read the last key (finite values
  // whose scores are masked).
  auto dma = [&](const char* base, const uint32_t (&go)[NDMA], bool is_v, int at, int sub, uint16_t* dst) {
    const char* blk = base + static_cast<int64_t>(static_cast<uint32_t>(at)) * kSub * stride_b;
    const int key0 = sub * kSub;
    if (key0 + kSub <= g.kv_len) {
#pragma unroll
      for (int c = 0; c < NDMA; ++c) dma16(blk + go[c], dst + 4 * (c * WAVES + wave) * kDim);
    } else {
#pragma unroll
      for (int c = 0; c < NDMA; ++c) {
        const int ra = 4 * (c * WAVES + wave) + (lane >> 4);
        const int rr = min(ra, g.kv_len - 1 - key0);
        const uint32_t off = rr * stride_b + 16 * (is_v ? v_seg(ra, lane & 15) : k_seg(ra, lane & 15));
        dma16(blk + off, dst + 4 * (c * WAVES + wave) * kDim);
      }
    }
  };
  // The same through registers for E4M3: whole 128-byte rows, 16 codes per
  // lane; stored widened to bf16.
  u32x4 rk[NRAW], rv[NRAW];
  auto fetch = [&](const char* base, int at, int sub, u32x4 (&dst)[NRAW]) {
    const char* blk = base + static_cast<int64_t>(static_cast<uint32_t>(at)) * kSub * stride_b;
#pragma unroll
    for (int i = 0; i < NRAW; ++i) {
      const int c = threadIdx.x + kThreads * i;
      const int rr = min(c >> 3, g.kv_len - 1 - sub * kSub);
      dst[i] = *reinterpret_cast<const u32x4*>(blk + rr * stride_b + 16 * (c & 7));
    }
  };
  auto store = [&](const u32x4 (&src)[NRAW], bool is_v, uint16_t* dst) {
#pragma unroll
    for (int i = 0; i < NRAW; ++i) {
      const int c = threadIdx.x + kThreads * i;
      const int ra = c >> 3;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int seg = 2 * (c & 7) + e;
        *reinterpret_cast<u32x4*>(dst + ra * kDim + 8 * (is_v ? v_seg(ra, seg) : k_seg(ra, seg))) =
            widen(u32x2{src[i][2 * e], src[i][2 * e + 1]});
      }
    }
  };

  // visited sub-blocks b + 1 .. b + 3 of iteration b: place (key row / 64) and
  // index, wave-uniform; and whether (which rows of) this wave selected b + 1
  auto place = [&](int i) -> int {
    if constexpr (SPARSE) return __builtin_amdgcn_readfirstlane(static_cast<int>(vis.at[min(i, nvisit - 1)]));
    else return i;
  };
  auto index = [&](int i) -> int {
    if constexpr (SPARSE) return __builtin_amdgcn_readfirstlane(static_cast<int>(vis.sub[min(i, nvisit - 1)]));
    else return i;
  };
  auto rows_of = [&](int sub) -> uint32_t {
    if constexpr (SPARSE)
      return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(vis.rows[wave][sub / SUB])));
    else
      return ~0u;
  };
  bf16x8 bq[KS];
  f32x16 acc_o[kDim / 32];
#pragma unroll
  for (int i = 0; i < kDim / 32; ++i) acc_o[i] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;
  // P of the pending sub-block in bf16, as the B operand of O^T = V^T P^T:
  // k-step u covers keys 32(u/2) + 16(u%2) + {4h + e, 8 + 4h + e}, e = 0..3
  bf16x8 bp[kSub / 16];
  float alpha_pend = 0.f;                 // alpha of the sub-block whose P is in bp

  // S^T = K Q^T on one sub-block: lane (n, h) gets keys 32i + 8(e/4) + 4h + e%4
  // of row n.  16 MFMA slots, each fenced off from the next so that the
  // compiler keeps the order; LDS operands are read kAhead slots ahead.
  auto scores = [&](const uint16_t* kbuf, f32x16 (&acc_s)[MT]) {
    const char* kbb = reinterpret_cast<const char*>(kbuf);
    constexpr int NS = MT * KS;
    auto kread = [&](int j) -> bf16x8 {
      return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(kbb + lo.ks[j % KS] + 2 * 32 * (j / KS) * kDim));
    };
#pragma unroll
    for (int i = 0; i < MT; ++i) acc_s[i] = f32x16{};
    bf16x8 kr[NS];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) kr[j] = kread(j);
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      if (j + kAhead < NS) kr[j + kAhead] = kread(j + kAhead);
      acc_s[j / KS] = mfma32x32x16(kr[j], bq[j % KS], acc_s[j / KS]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // sum of eight weights: of their rounded values (dense) or as they are
  auto add_weights = [&](float lsum, const f32x16& a, int e0, const uint4& pw) -> float {
    if constexpr (SPARSE) {
#pragma unroll
      for (int e = 0; e < 8; ++e) lsum += a[e0 + e];
      return lsum;
    } else {
      return add_bf16_pair(add_bf16_pair(add_bf16_pair(add_bf16_pair(lsum, pw.x), pw.y), pw.z), pw.w);
    }
  };

  // online softmax of one sub-block's scores (raw units; scale_log2 > 0 keeps
  // the order): updates m_run / l_run, leaves P in bp, returns alpha
  auto softmax = [&](f32x16 (&acc_s)[MT], int key0, bool sel, auto masked) -> float {
    if constexpr (decltype(masked)::value) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = key0 + 32 * i + 8 * (e >> 2) + 4 * h + (e & 3);
          acc_s[i][e] = key <= p ? acc_s[i][e] : -INFINITY;
        }
    }
    float bmax = -INFINITY;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) bmax = fmaxf(bmax, acc_s[i][e]);
    bmax = fmaxf(bmax, xor32f(bmax));
    if (SPARSE) bmax = sel ? bmax : -INFINITY;
    const float m_new = fmaxf(m_run, bmax);
    const float mm = m_new == -INFINITY ? 0.f : m_new;     // rows with nothing visible yet
    const float alpha = exp2_hw((m_run - mm) * scale_log2);
    const float neg = SPARSE && !sel ? -INFINITY : -mm * scale_log2;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float w = exp2_hw(fmaf(acc_s[i][e], scale_log2, neg));
        acc_s[i][e] = !SPARSE || sel ? w : 0.f;
      }
    float lsum = 0.f;
#pragma unroll
    for (int u = 0; u < kSub / 16; ++u) {
      uint4 pw;
      const int i = u >> 1, e0 = 8 * (u & 1);
      pw.x = pack_bf16x2(acc_s[i][e0 + 0], acc_s[i][e0 + 1]);
      pw.y = pack_bf16x2(acc_s[i][e0 + 2], acc_s[i][e0 + 3]);
      pw.z = pack_bf16x2(acc_s[i][e0 + 4], acc_s[i][e0 + 5]);
      pw.w = pack_bf16x2(acc_s[i][e0 + 6], acc_s[i][e0 + 7]);
      lsum = add_weights(lsum, acc_s[i], e0, pw);
      bp[u] = __builtin_bit_cast(bf16x8, pw);
    }
    lsum += xor32f(lsum);
    l_run = l_run * alpha + lsum;
    m_run = m_new;
    return alpha;
  };

  // O is rescaled by the pending sub-block's alpha only when some row's maximum moved
  auto rescale = [&]() {
    if (__ballot(alpha_pend != 1.f)) {
#pragma unroll
      for (int i = 0; i < kDim / 32; ++i) acc_o[i] *= alpha_pend;
    }
  };
  // V^T operand of k-step u, dim tile td, read down V's columns
  auto read_vt = [&](const uint16_t* vbuf, int u, int td) -> bf16x8 {
    const char* a0 = reinterpret_cast<const char*>(vbuf) + lo.vs[td] + 2 * (32 * (u >> 1) + 16 * (u & 1)) * kDim;
    const uint2 x0 = lds_tr4(reinterpret_cast<const uint16_t*>(a0));
    const uint2 x1 = lds_tr4(reinterpret_cast<const uint16_t*>(a0 + 2 * 8 * kDim));  // rows +8: same permutation
    return __builtin_bit_cast(bf16x8, make_uint4(x0.x, x0.y, x1.x, x1.y));
  };
  // O^T += V^T P^T from one value sub-block in 16 fenced MFMA slots, beside(j)
  // after the j-th
  auto pv = [&](const uint16_t* vbuf, auto beside) {
    constexpr int NO = (kSub / 16) * (kDim / 32);
    auto vread = [&](int j) { return read_vt(vbuf, j / (kDim / 32), j % (kDim / 32)); };
    bf16x8 vr[NO];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) vr[j] = vread(j);
#pragma unroll
    for (int j = 0; j < NO; ++j) {
      if (j + kAhead < NO) vr[j + kAhead] = vread(j + kAhead);
      acc_o[j % (kDim / 32)] = mfma32x32x16(vr[j], bp[j / (kDim / 32)], acc_o[j % (kDim / 32)]);
      beside(j);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto nothing = [](int) {};

  // iteration b: K_{b+1} is in k[(b+1)&1], V_b in v[b&1]; after the S^T slots
  // each O^T slot carries one sixteenth of the next softmax, so the VALU works
  // while the MFMA pipe drains.
  int at1 = 0, at2 = 0, at3 = 0, sub1 = 0, sub2 = 0, sub3 = 0;
  uint32_t word1 = ~0u;
  auto step = [&](int b, auto masked_t) {
    constexpr bool masked = decltype(masked_t)::value;
    __builtin_amdgcn_s_waitcnt(0);        // this thread's copies of K_{b+1} and V_b have landed
    __syncthreads();                      // everyone's have, and block b-1's readers are done
    if constexpr (!SPARSE) {              // sub-block i is at key 64 i: nothing carried from step to step
      if (b + 2 < nvisit) dma(kb, lo.kg, false, b + 2, b + 2, ring.k[b & 1]);
      dma(vb, lo.vg, true, b + 1, b + 1, ring.v[(b + 1) & 1]);
    } else if constexpr (kDma) {
      if (b + 2 < nvisit) dma(kb, lo.kg, false, at2, sub2, ring.k[b & 1]);
      dma(vb, lo.vg, true, at1, sub1, ring.v[(b + 1) & 1]);
    } else {
      if (b + 2 < nvisit) store(rk, false, ring.k[b & 1]);
      store(rv, true, ring.v[(b + 1) & 1]);
      if (b + 3 < nvisit) fetch(kb, at3, sub3, rk);
      if (b + 2 < nvisit) fetch(vb, at2, sub2, rv);
    }
    const int key0 = (SPARSE ? sub1 : b + 1) * kSub;
    const bool sel = !SPARSE || ((word1 >> jq) & 1u);
    if constexpr (SPARSE) {
      at1 = at2; sub1 = sub2; at2 = at3; sub2 = sub3;
      at3 = place(b + 4);
      sub3 = index(b + 4);
      word1 = rows_of(sub1);
    }
    rescale();
    __builtin_amdgcn_sched_barrier(0);
    f32x16 acc_s[MT];
    scores(ring.k[(b + 1) & 1], acc_s);
    bf16x8 bp_next[kSub / 16];
    float m0 = -INFINITY, m_new = 0.f, alpha = 0.f, neg = 0.f, lsum = 0.f;
    pv(ring.v[b & 1], [&](int j) __attribute__((always_inline)) {
      if (j == 0) {
        if constexpr (masked) {
#pragma unroll
          for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const int key = key0 + 32 * i + 8 * (e >> 2) + 4 * h + (e & 3);
              acc_s[i][e] = key <= p ? acc_s[i][e] : -INFINITY;
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) m0 = fmaxf(m0, acc_s[0][e]);
      } else if (j == 1) {
#pragma unroll
        for (int e = 0; e < 16; ++e) m0 = fmaxf(m0, acc_s[1][e]);
        m0 = fmaxf(m0, xor32f(m0));
        if (SPARSE) m0 = sel ? m0 : -INFINITY;
        m_new = fmaxf(m_run, m0);
        const float mm = m_new == -INFINITY ? 0.f : m_new;   // rows with nothing visible yet
        alpha = exp2_hw((m_run - mm) * scale_log2);
        neg = SPARSE && !sel ? -INFINITY : -mm * scale_log2;
      } else if (j < 14) {
#pragma unroll
        for (int x = 0; x < 32; ++x) {
          if (2 + (3 * x) / 8 != j) continue;
          acc_s[x >> 4][x & 15] = exp2_hw(fmaf(acc_s[x >> 4][x & 15], scale_log2, neg));
        }
      } else {
#pragma unroll
        for (int u = 2 * (j - 14); u < 2 * (j - 14) + 2; ++u) {
          uint4 pw;
          const int i = u >> 1, e0 = 8 * (u & 1);
          pw.x = pack_bf16x2(acc_s[i][e0 + 0], acc_s[i][e0 + 1]);
          pw.y = pack_bf16x2(acc_s[i][e0 + 2], acc_s[i][e0 + 3]);
          pw.z = pack_bf16x2(acc_s[i][e0 + 4], acc_s[i][e0 + 5]);
          pw.w = pack_bf16x2(acc_s[i][e0 + 6], acc_s[i][e0 + 7]);
          lsum = add_weights(lsum, acc_s[i], e0, pw);
          bp_next[u] = __builtin_bit_cast(bf16x8, pw);
        }
        if (j == 15) {
          lsum += xor32f(lsum);
          l_run = l_run * alpha + lsum;
          m_run = m_new;
        }
      }
    });
#pragma unroll
    for (int u = 0; u < kSub / 16; ++u) bp[u] = bp_next[u];
    alpha_pend = alpha;
  };

  auto write_rows = [&]() {
    if (!valid) return;
    const bool empty = !(l_run > 0.f);
    const float inv_l = empty ? 0.f : o_scale / l_run;
    // O^T tile td: lane (n, h) holds d = 32td + 8(e/4) + 4h + e%4 of row n
    uint16_t* orow = o + head_row * kDim + 4 * h;
#pragma unroll
    for (int td = 0; td < kDim / 32; ++td)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        uint2 w;
        w.x = pack_bf16x2(acc_o[td][4 * e4 + 0] * inv_l, acc_o[td][4 * e4 + 1] * inv_l);
        w.y = pack_bf16x2(acc_o[td][4 * e4 + 2] * inv_l, acc_o[td][4 * e4 + 3] * inv_l);
        *reinterpret_cast<uint2*>(orow + 32 * td + 8 * e4) = w;
      }
    if (h == 0) lse[head_row] = empty ? -INFINITY : (m_run * scale_log2 + __log2f(l_run)) * kLn_2;
  };

  if (nvisit > 0) {
    const int at0 = place(0), sub0 = index(0);
    at1 = place(1); sub1 = index(1);
    at2 = place(2); sub2 = index(2);
    at3 = place(3); sub3 = index(3);
    const uint32_t word0 = rows_of(sub0);
    word1 = rows_of(sub1);
    if constexpr (kDma) {
      dma(kb, lo.kg, false, at0, sub0, ring.k[0]);
      dma(vb, lo.vg, true, at0, sub0, ring.v[0]);
      if (nvisit > 1) dma(kb, lo.kg, false, at1, sub1, ring.k[1]);
    } else {
      u32x4 r0[NRAW], r1[NRAW], r2[NRAW];
      fetch(kb, at0, sub0, r0);
      fetch(vb, at0, sub0, r1);
      if (nvisit > 1) fetch(kb, at1, sub1, r2);
      if (nvisit > 2) fetch(kb, at2, sub2, rk);
      if (nvisit > 1) fetch(vb, at1, sub1, rv);
      store(r0, false, ring.k[0]);
      store(r1, true, ring.v[0]);
      if (nvisit > 1) store(r2, false, ring.k[1]);
    }
#pragma unroll
    for (int st = 0; st < KS; ++st) bq[st] = __builtin_bit_cast(bf16x8, widen(rq[st]) ^ q_flip);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    {
      f32x16 acc_s[MT];
      scores(ring.k[0], acc_s);
      const bool sel = !SPARSE || ((word0 >> jq) & 1u);
      alpha_pend = sub0 < nfree ? softmax(acc_s, 0, sel, std::false_type{}) : softmax(acc_s, sub0 * kSub, sel, std::true_type{});
    }
    int b = 0;
    if constexpr (SPARSE) {
      for (; b + 1 < nvisit && sub1 < nfree; ++b) step(b, std::false_type{});
    } else {
      for (; b + 1 < min(nfree, nvisit); ++b) step(b, std::false_type{});
    }
    for (; b + 1 < nvisit; ++b) step(b, std::true_type{});
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    rescale();
    pv(ring.v[b & 1], nothing);
  }
  write_rows();                             // (before the check: the stores go out beside it)
  if constexpr (SPARSE) {
    if (nvisit > 0) {
      float zero[kDim / 32];                // NaN unless everything is finite
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int i = 0; i < kDim / 32; ++i) zero[i] = fmaf(acc_o[i][e], 0.f, e == 0 ? l_run * 0.f : zero[i]);
      if (__ballot(zero[0] + zero[1] + zero[2] + zero[3] != 0.f) && lane == 0) vis.redo = 1;
      __syncthreads();
      if (vis.redo != 0) {                  // uniform over the CTA
#pragma unroll
        for (int i = 0; i < kDim / 32; ++i) acc_o[i] = f32x16{};
        m_run = -INFINITY;
        l_run = 0.f;
#pragma unroll 1
        for (int i = 0; i < nvisit; ++i) {
          const int at = place(i), sub = index(i);
          const bool sel = (rows_of(sub) >> jq) & 1u;
          __syncthreads();                  // the previous sub-block's readers are done
          if constexpr (kDma) {
            dma(kb, lo.kg, false, at, sub, ring.k[0]);
            dma(vb, lo.vg, true, at, sub, ring.v[0]);
          } else {
            fetch(kb, at, sub, rk);
            store(rk, false, ring.k[0]);
            fetch(vb, at, sub, rk);
            store(rk, true, ring.v[0]);
          }
          __builtin_amdgcn_s_waitcnt(0);
          __syncthreads();
          f32x16 acc_s[MT];
          scores(ring.k[0], acc_s);
          const float alpha = softmax(acc_s, sub * kSub, sel, std::true_type{});
#pragma unroll
          for (int td = 0; td < kDim / 32; ++td) {
            f32x16 d = acc_o[td] * alpha;
#pragma unroll
            for (int u = 0; u < kSub / 16; ++u) d = mfma32x32x16(read_vt(ring.v[0], u, td), bp[u], d);
#pragma unroll
            for (int e = 0; e < 16; ++e) acc_o[td][e] = sel ? d[e] : acc_o[td][e];
          }
        }
        write_rows();
      }
    }
  }
}

}  // namespace flash
}  // namespace
