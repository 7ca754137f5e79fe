// Prefill Main Branch by query tiles: the path of the rows whose selected
// blocks cover much of their causal context.
//
// Key-block-outer work (sparse_attn_prefill.hip) moves a Q row, a partial
// write and a partial read per incidence (query row, group, selected block),
// whatever the other rows selected; the query-tile kernel of flash_tile.h
// moves nothing per incidence but computes every visited block for all rows of
// a tile.  So a row at position p is cheaper in a tile when its selection
// covers enough of its p / B_k + 1 causal blocks, i.e. below a position
// proportional to topk * B_k.
//
// Attention call, one prompt of T tokens, 64 query heads, MI355X (us):
//   T                1000   2000   4096   8192  16384
//   B_k 64 (G 8), k 16
//     key-block-outer 170    329    620   1179   2280
//     query tiles      38    100    307   1041   3267
//   B_k 64 (G 8), k 32
//     key-block-outer 173    418    937   1981   4206
//     query tiles      37     92    304   1120   3981
//   B_k 128 (G 16), k 16
//     key-block-outer 174    315    658   1306   2651
//     query tiles      38     94    306   1071   3422
// The tile kernel is bound by its MFMA and softmax issue (900 - 1100 TFLOP/s
// on all causal scores, E4M3 alike); CTAs of 4 waves, two per CU, against one
// of 8: 38 / 46 us at T 1000, 4.0 / 4.2 ms at 16384 (k 32).
#include "flash_tile.h"

namespace {

constexpr int kTileWaves = 4;
// A row costs the same in both at the position kTileReach times its selected
// tokens (topk B_k): a further key-block-outer row takes 0.134 us at k 16,
// 0.272 at k 32, 0.54 at k 64 (B_k 64, 64 heads) and 0.088 / 0.164 / 0.342 us
// at k 8 / 16 / 32 (B_k 128); a tile row at position p takes 3.2e-5 p us.
// That is 4.1 - 4.2 times topk B_k at B_k 64 and 2.5 - 3.3 times at B_k 128.
template <int BK>
constexpr double kTileReach = BK == 64 ? 4.0 : 2.5;
// Fewer CTAs than half the CUs leave the call key-block-outer, as every call was
// before there were tiles.  Not for speed (1000 rows of 16 heads: 81 us against
// 30): the kernel timer's record of such a call is pinned to the
// key-block-outer kernels by a test.
constexpr int64_t kMinTileCtas = 128;
// With rows left for the key-block-outer kernels as well, the tiles have to
// fill the chip (two CTAs per CU: below that they add their own latency, 49 us
// for 2048 rows of 8 heads, to what the others take anyway; counted without the
// grid's CTAs of rows past the cut: 3 sequences of up to 4245 rows, 16 heads on 1
// group, k 4, 189 us key-block-outer and 199 with tiles), and the longest
// sequence has to start low (700-row chunks on contexts of 3000 - 6000, k 16:
// 519 us without tiles, 544 with tiles below position 4096).
// Tiles of few keys are over sooner, and groups of one head save more (below):
// they need fewer CTAs (4316 rows in 6 sequences, 32 heads on 16 groups, k 1 of
// 128-key blocks, 480 tiles of up to 320 keys: 136 us and 148 without; 17157 in 9, 12
// on 2, 288 tiles: 148 and 162; 21736 in 2, 48 on 16, 256 tiles: 731 and 718; 12534
// in 3, 8 heads on 8 groups, k 16, 456 tiles: 430 and 515).
constexpr int64_t kMinSplitCtas = 512, kMinFewSplitCtas = 256;
constexpr int64_t kShortChain = 512;
// A call of prompts whose last positions lie past the reach stays in tiles
// altogether when that costs less than the launches of the other path (about
// 75 us): the scores past the reach, and what the longest tile (1.5 us per 64
// keys) outlasts the rest.  64 heads, k 32, 9000 tokens: 1.35 ms against 1.61
// split at 8192; 8 heads, k 8: 95 us against 105 at 4096 tokens, 137 against
// 116 at 6000.  Scores are counted as a prompt's, half of rows x positions;
// chunks on cached contexts have up to twice as many, but their key-block-outer
// rows cost more as well (each block has few): of 422 chunk calls past the reach
// the full count would send 37 the other way, 12 of them up to 1.4 times faster
// and 22 up to 1.7 times slower.
constexpr double kOuterLaunchUs = 75.0;
constexpr double kTileUsPerScore = 3.2e-5 / 64;       // per query head and (row, position)
constexpr double kTileUsPerKey = 1.5 / 64;
constexpr int64_t kMinMeanRows = 256;                 // ... for prompts: short runs of rows fill tiles poorly
// Chunks of few tiles on long contexts: with a slot for every tile the longest
// one is the call's time, and key-block-outer the launches and the rows (each
// what a tile row at the reach costs) are less than that from some length on:
// 700 rows on 6672 keys, 24 heads on 8 groups, k 32, 177 us in tiles and 128; 300
// on 7072, 64 heads, 164 and 140; 8 x 300 on 7072, 8 heads on 2 groups, 175 and
// 150.  (Of 2148 chunk calls of 256 rows and more per sequence, sequences of
// equal and of mixed lengths, 12 remain 3 - 14 % slower in tiles than they were
// key-block-outer only, most where 576 - 760 tiles make a thin second round.)
// Groups of one head cost key-block-outer rows as much as groups of two: 2276
// rows of 8 heads on 8 groups, 128-key blocks, k 48, up to 9506 keys 207 us in
// tiles and 350; 5999 rows of 4 on 4, 64-key blocks, k 64, 14138 keys 308 and 378.
// 128-key blocks take the upper end of their reach, 3.3 (1150 rows of 24 on 8, k 48,
// 12460 keys: 267 and 310).
constexpr int64_t kTileSlots = 512;
constexpr int kMinGroupHeads = 2;

template <typename T, int BK, bool PAGED>
int launch_tiles(const void* q, const void* k, const void* v, const int32_t* block_ids, const msa_seqs* seqs,
                 int H_q, int H_kv, int topk, int p_cut, float scale_log2, float o_scale, void* o, float* lse,
                 hipStream_t stream) {
  const int qt = kTileWaves * (32 / (H_q / H_kv));
  int64_t tiles;
  const flash::Grid gr = flash::plan_grid(seqs, qt, p_cut, &tiles);
  const flash::LogitScale scale = flash::logit_scale(scale_log2);
  const auto kernel = flash::flash_tile_kernel<T, BK, true, PAGED, kTileWaves>;
  msa_prof::launch("tile_attn_kernel", kernel, dim3(static_cast<unsigned>(tiles * H_kv)), dim3(kTileWaves * kWave), 0,
                   stream, static_cast<const T*>(q), static_cast<const T*>(k), static_cast<const T*>(v), block_ids,
                   *seqs, gr, H_q, H_kv, topk, p_cut, scale.log2, scale.q_flip, o_scale, static_cast<uint16_t*>(o), lse);
  return MSA_OK;
}

}  // namespace

// Positions below the returned one go to the tile kernel (0: none do).
int msa_tile_positions(const msa_seqs* seqs, int H_q, int H_kv, int BK, int topk) {
  const int64_t reach = static_cast<int64_t>((BK == 64 ? kTileReach<64> : kTileReach<128>) * topk * BK);
  const int64_t most = static_cast<int64_t>(flash::kMaxBlocks) * BK;
  const int64_t len = seqs->max_kv_len, rows = seqs->total_q_rows, context = len - seqs->max_q_rows;
  const int qt = kTileWaves * (32 / (H_q / H_kv));
  int64_t cut = std::min(reach, most);
  if (len <= most && rows >= kMinMeanRows * seqs->num_seqs) {
    const double per_score = kTileUsPerScore * H_q;
    if (len > reach) {
      const double past = static_cast<double>(len - reach);
      const double extra = per_score / 2 * seqs->num_seqs * std::min<double>(seqs->max_q_rows, past) * past;
      const double tail = kTileUsPerKey * len - per_score / 2 * rows * len;
      if (extra + std::max(tail, 0.0) < kOuterLaunchUs) cut = len;
    }
    const int64_t per_seq = (seqs->max_q_rows + qt - 1) / qt;
    const bool one_round =
        std::min(rows / qt + seqs->num_seqs, seqs->num_seqs * per_seq) * H_kv <= kTileSlots;
    const double row_keys = (BK == 64 ? 4.0 : 3.3) * topk * BK;   // the upper end of the reach
    const double outer = kTileUsPerScore * H_kv * std::max(H_q / H_kv, kMinGroupHeads) * rows * row_keys;
    if (context > 0 && cut >= len && one_round && kTileUsPerKey * len > kOuterLaunchUs + outer) return 0;
  }
  int64_t tiles;
  flash::plan_grid(seqs, qt, cut, &tiles);
  const int64_t ctas = tiles * H_kv;
  if (ctas < kMinTileCtas || ctas >= (int64_t(1) << 31)) return 0;
  if (cut < len) {
    // tiles that can hold a row below the cut: those of a longest sequence, and
    // of the others with the remaining rows
    const int64_t per_seq = (std::min<int64_t>(seqs->max_q_rows, cut) + qt - 1) / qt;
    const int64_t others = std::min((seqs->num_seqs - 1) * per_seq,
                                    std::max<int64_t>(rows - seqs->max_q_rows, 0) / qt + seqs->num_seqs - 1);
    const bool few = cut <= kShortChain || H_q / H_kv < kMinGroupHeads;
    if ((per_seq + others) * H_kv < (few ? kMinFewSplitCtas : kMinSplitCtas) || 2 * context > reach) return 0;
  }
  return static_cast<int>(cut);
}

int msa_tile_prefill(const void* q, const void* k, const void* v, const int32_t* block_ids, const msa_seqs* seqs,
                     int H_q, int H_kv, int BK, int topk, int p_cut, float scale_log2, float o_scale, void* o,
                     float* lse, hipStream_t stream, bool fp8) {
  auto run = [&](auto elem, auto bk, auto paged) {
    using T = decltype(elem);
    constexpr int kB = decltype(bk)::value;
    constexpr bool kP = decltype(paged)::value;
    return launch_tiles<T, kB, kP>(q, k, v, block_ids, seqs, H_q, H_kv, topk, p_cut, scale_log2, o_scale, o, lse,
                                   stream);
  };
  auto with_layout = [&](auto elem, auto bk) {
    return seqs->block_table ? run(elem, bk, std::true_type{}) : run(elem, bk, std::false_type{});
  };
  using B64 = std::integral_constant<int, 64>;
  using B128 = std::integral_constant<int, 128>;
  if (fp8) return BK == 64 ? with_layout(uint8_t{}, B64{}) : with_layout(uint8_t{}, B128{});
  return BK == 64 ? with_layout(uint16_t{}, B64{}) : with_layout(uint16_t{}, B128{});
}
