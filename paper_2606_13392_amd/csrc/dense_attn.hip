// Dense causal GQA attention on gfx950: the baseline the sparse path is
// measured against.  Every query attends to all causally visible keys of its
// sequence (the full-attention form that MSA's sparse-attention equation of
// Sec. 3.1 reduces to when k covers every causal block), with the layout
// conventions of the sparse calls.
//
// Prefill runs the query-tile kernel of flash_tile.h over every causal key
// block: 8 waves of 32 (query row, head) rows per CTA, one CTA per CU.
//
// Decode (at most four query rows per sequence) runs the row kernel of the
// sparse decode call over every key block (msa_rows_dense).
#include "flash_tile.h"

// every key block of each row, split over waves and CTAs (sparse_attn.hip)
size_t msa_rows_dense_workspace_size(const msa_seqs* seqs, int H_q, int H_kv);
int msa_rows_dense(const void* q, const void* k, const void* v, const msa_seqs* seqs, int H_q, int H_kv,
                   float scale, void* o, float* lse, void* workspace, size_t workspace_bytes, hipStream_t stream);

namespace {

using namespace msa;

constexpr int kHeadDim = flash::kDim;
constexpr float kLog2e = flash::kLog2E;
constexpr int kDecodeRows = 4;           // sequences with at most this many query rows take the row kernel
constexpr int kWaves = 8;                // waves per CTA (32 MFMA rows each), one CTA per CU

int validate_dense(const msa_seqs* seqs, int H_q, int H_kv, int head_dim) {
  int st = msa_host::validate_seqs(seqs);
  if (st != MSA_OK) return st;
  if (H_q < 1 || H_kv < 1 || head_dim < 1 || H_q % H_kv != 0) return MSA_ERR_INVALID;
  if (head_dim != kHeadDim) return MSA_ERR_UNSUPPORTED;
  if (H_q / H_kv > 16 || H_kv > 64) return MSA_ERR_UNSUPPORTED;
  if (seqs->total_q_rows * H_kv >= (int64_t(1) << 31)) return MSA_ERR_UNSUPPORTED;
  if (seqs->block_table) return MSA_ERR_UNSUPPORTED;   // contiguous key side only
  return MSA_OK;
}

bool decode_like(const msa_seqs* seqs) { return seqs->max_q_rows <= kDecodeRows; }

}  // namespace

extern "C" size_t msa_dense_attn_workspace_size(const msa_seqs* seqs, int num_q_heads, int num_kv_heads,
                                               int head_dim) {
  if (validate_dense(seqs, num_q_heads, num_kv_heads, head_dim) != MSA_OK) return 0;
  if (decode_like(seqs)) return msa_rows_dense_workspace_size(seqs, num_q_heads, num_kv_heads);
  // not read or written; part of the call's contract since it held a tile table
  return msa_host::align_up(sizeof(int32_t) * (seqs->num_seqs + 1), 256);
}

extern "C" int msa_dense_attn(const void* q, const void* k, const void* v, const msa_seqs* seqs, int num_q_heads,
                              int num_kv_heads, int head_dim, float softmax_scale, void* o, float* lse,
                              void* workspace, size_t workspace_bytes, hipStream_t stream) {
  int st = validate_dense(seqs, num_q_heads, num_kv_heads, head_dim);
  if (st != MSA_OK) return st;
  if (seqs->total_q_rows == 0) return MSA_OK;
  if (!q || !k || !v || !o || !lse) return MSA_ERR_INVALID;
  const flash::LogitScale scale = flash::logit_scale(softmax_scale * kLog2e);
  if (decode_like(seqs))
    return msa_rows_dense(q, k, v, seqs, num_q_heads, num_kv_heads, softmax_scale, o, lse, workspace,
                          workspace_bytes, stream);
  const size_t need = msa_host::align_up(sizeof(int32_t) * (seqs->num_seqs + 1), 256);
  if (!workspace || workspace_bytes < need) return MSA_ERR_WORKSPACE;
  const int G = num_q_heads / num_kv_heads;
  const int qt = kWaves * (32 / G);
  int64_t tiles;
  flash::Grid gr = flash::plan_grid(seqs, qt, seqs->max_q_rows, &tiles);
  gr.tile_fast = flash::tile_fast(seqs, num_kv_heads, qt);
  if (tiles * num_kv_heads >= (int64_t(1) << 31)) return MSA_ERR_UNSUPPORTED;
  const auto kernel = flash::flash_tile_kernel<uint16_t, 64, false, false, kWaves>;
  msa_prof::launch("dense_prefill_kernel", kernel, dim3(static_cast<unsigned>(tiles * num_kv_heads)),
                   dim3(kWaves * kWave), 0, stream, static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k),
                   static_cast<const uint16_t*>(v), static_cast<const int32_t*>(nullptr), *seqs, gr, num_q_heads,
                   num_kv_heads, 0, 0, scale.log2, scale.q_flip, 1.f, static_cast<uint16_t*>(o), lse);
  return msa_host::launch_status();
}
