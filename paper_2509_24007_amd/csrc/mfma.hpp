// Matrix-core (MFMA) kernels of the bf16 mode: declarations.
#pragma once
#include "internal.hpp"

namespace sdlm {

// True when the bf16 matrix-core path serves this model (bf16, head_dim 128, sizes multiples of the tile steps).
bool mfma_supported(const sdlm_model_cfg *m);
// Rows of a packed weight matrix are padded to a multiple of the 32-row tile.
size_t mfma_pad_n(size_t N);
// Elements a packed [N, K] matrix occupies (N * K when `packed` is false).
size_t mfma_packed_elems(bool packed, size_t N, size_t K);
// Bytes of scratch the split-KV attention needs for its per-chunk partial results.
size_t mfma_attn_scratch_bytes(const sdlm_model_cfg *m, const sdlm_run_cfg *r, int max_rows);
// Bytes of scratch for the LM head's per-vocabulary-block partials.
size_t mfma_lm_scratch_bytes(int V, int max_rows);
// Smallest KV chunk (in 16-key tiles) the attention launch over `groups` row groups may use with this much scratch.
int mfma_attn_chunk_floor(const sdlm_model_cfg *m, int max_seq_len, int groups, size_t scratch_bytes);
// Rows of one sequence that form one attention work item (rows x query heads per kv head <= 64).
int mfma_group_rows(const sdlm_model_cfg *m);

// Repack rows of a row-major [N, K] bf16 matrix into tile order at row offset dst_row0 of a packed matrix with
// dst_rows rows.  interleave: 0 plain; 1 / 2: the matrix is the gate / up half of the fused gate-up matrix,
// whose 32-row tiles alternate gate, up.
void launch_pack_mfma(hipStream_t s, void *dst, const void *src, int N, int K, int dst_row0, int dst_rows, int interleave);
// The launch shape launch_gemm_mfma takes (host logic only): rows and columns of a workgroup's tile and number of k splits.  Columns are
// those of the packed matrix (for gate/up, EPI_SWIGLU, the fused one of 2N rows).
void mfma_gemm_plan(int epi, int rows, int min_rows, int N, int K, size_t slab_room_floats, int *tile_rows, int *tile_cols, int *splits);
// Returns the number of split-k slabs written to `slabs` (1: the result is complete in a.Yf / a.Yt).  For
// EPI_STORE_F32 the consumer always adds the slabs; for EPI_RESID the slabs are added to a.Yf here unless
// defer_reduce, in which case the next RMSNorm adds them (slab stride = a.max_rows * a.N floats).
int launch_gemm_mfma(hipStream_t s, int epi, const GemmArgs &a, float *slabs, size_t slab_room_floats, bool defer_reduce);
// part 0: the attention kernel; part 1: the merge of the split-KV partials (a no-op when the launch has a single
// chunk).  Returns whether the launch shape needs the merge.  max_seq_len: capacity, which sizes the launch; max_len: upper bound of the
// sequences' present lengths, which together with the row groups decides the form of the launches (mfma_attn_form).  two_staging: row groups of this pass may read a second
// staging tile (a verification pass whose rows do not fit one tile).
bool launch_attn_mfma(hipStream_t s, const sdlm_model_cfg *m, int max_seq_len, int max_len, const void *q, void *out, const void *pool_layer,
                      const KvGeom &kg, const RowMeta &rm, const SeqState &st, int D, int max_groups, void *scratch, size_t scratch_bytes,
                      int part, bool two_staging);
// That form, a small integer: a captured pass may be replayed while it stays the same.
int mfma_attn_form(const sdlm_model_cfg *m, int max_seq_len, int max_len, int max_groups, size_t scratch_bytes, bool two_staging);
// Steps of at most 32 rows, and of more where qkv_rope_skinny_applies: QKV projection, rotation and K/V placement in one launch (same results as the projection
// followed by the RoPE + K/V placement kernel, up to the order in which the k partial sums are added).
bool qkv_rope_skinny_applies(const sdlm_model_cfg *m, int max_rows, int min_rows);   // min_rows: rows that are certainly there
void mfma_qkv_rows(const sdlm_model_cfg *m, int max_rows, int min_rows, int *rows, int *rest_rows);   // rows of a block that certainly holds some and of one that may be empty (0: not in one launch)
void launch_qkv_rope_skinny(hipStream_t s, const sdlm_model_cfg *m, const void *X, const void *w_packed, const void *bias, const int32_t *p_rows,
                            int max_rows, int min_rows, void *q_out, void *pool_layer, const KvGeom &kg, const RowMeta &rm, const SeqState &st, const float2 *rope,
                            const float *ssq = nullptr, float eps = 0.f);
// Steps of at most 16 rows: norms inside the products.  The rows' operand `xg` (16 x h bf16: x times the gains of the coming norm, in the matrix instruction's order)
// and their sums of squares `ssq` ([16][h / 16] floats) are left by the embedding and by O and down, and read by the fused QKV launch (which then gets ssq) and by
// gate/up; gate/up leaves its result in that order too, which down reads (`ordered`).  gain: null where no layer follows.
bool mfma_few_applies(const sdlm_model_cfg *m, int max_rows);
void launch_embed_few(hipStream_t s, float *x, const void *E, const RowMeta &rm, int max_rows, int h, int V, const void *gain, void *xg, float *ssq);
void launch_gateup_few(hipStream_t s, const GemmArgs &g, const float *ssq, float eps);
void launch_resid_few(hipStream_t s, const GemmArgs &g, bool ordered, const void *gain, void *xg, float *ssq);
// Down of such a step: by launch_resid_few, or split along k with its sums left to an RMSNorm (defer_reduce and return value as in launch_gemm_mfma).
bool few_down_whole(int h);
int launch_down_split(hipStream_t s, const GemmArgs &g, float *slabs, size_t slab_room_floats, bool defer_reduce);
void launch_unorder(hipStream_t s, void *dst, const void *src, int rows, int K);   // an operand of that chain as rows (taps)
void launch_lmhead_mfma(hipStream_t s, const void *xhat, const void *w_packed, const int32_t *p_rows, int max_rows, int min_rows, int V, int h,
                        float scale, int conf_fn, float *logits_out, void *scratch, int32_t *ids, float *conf);

}  // namespace sdlm
