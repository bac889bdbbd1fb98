// Shape-generic kernels of the block-decode step: row assembly, embedding gather, RMSNorm, a tiled FMA GEMM with
// fused epilogues, RoPE + K/V placement, block-masked attention, the vocabulary reduction, prefix acceptance
// and commit.  Storage is fp32 or bf16; all arithmetic is fp32.  They serve the fp32 debug mode and every small
// integer/elementwise step of the bf16 mode; the bf16 mode's contractions run on the matrix-core kernels.
#include <type_traits>

#include "internal.hpp"

namespace sdlm {

// Embeddings of R rows by one workgroup, four features a thread.  One workgroup is enough while the gather is a few trips, each a round trip for the token and one for
// its row; it saves a launch of 2.4 us (h = 256, 8 rows: assembly and gather 5.2 -> 3.4 us; the rule of assemble_embeds).
template <typename T>
__device__ inline void embed_rows(float *x, const T *E, const int32_t *tok, int R, int h, int V)
{
    const int per = h / 4, n = R * per;   // h is a multiple of 4
    for (int e = threadIdx.x; e < n; e += blockDim.x) {
        const int r = e / per, k = e % per * 4;
        const T *src = E + (size_t)min(max(tok[r], 0), V - 1) * h + k;
        *(float4 *)(x + (size_t)r * h + k) = make_float4(to_f<T>(src[0]), to_f<T>(src[1]), to_f<T>(src[2]), to_f<T>(src[3]));
    }
}

// ------------------------------------------------------------------------------------------------ row assembly
// Rows of a decode step, per sequence: the pending tokens (positions c..n-1, causal), then the block
// [x_last, [m] x (D-1)] at positions n-1 .. n+D-2 (block definition, Sec. 3.2).  A block row may see the cache
// below position s = n-1 only; the causal copy of x_last at s is for later steps.
// E: embedding table (storage type T), gathered here into x for few rows (see launch_assemble_decode), else null.
template <typename T>
__global__ void assemble_decode_k(SeqState st, RowMeta rm, int B, int D, int mask_id, int gr, int stg0, int causal, int Hkv, int cp_floor, float *x, const T *E, int h, int V)
{
    __shared__ int row0[1025], grp0[1025], cp_s;
    if (threadIdx.x == 0) {
        int r = 0, g = 0;
        long tiles = 0;   // 16-key tiles the attention's work items stream, per kv head
        for (int b = 0; b < B; ++b) {
            row0[b] = r; grp0[b] = g;
            int rows = st.n[b] - st.c[b] + D, ng = (rows + gr - 1) / gr;
            r += rows;
            g += ng;
            tiles += (long)ng * ((st.n[b] + PAGE - 1) / PAGE);
        }
        row0[B] = r; grp0[B] = g;
        cp_s = attn_chunk_pages(tiles * Hkv, cp_floor);
        rm.counts[0] = r; rm.counts[1] = g; rm.counts[2] = B * D; rm.counts[3] = cp_s;
    }
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += blockDim.x) {
        int n = st.n[b], c = st.c[b], p = n - c, r = row0[b];
        for (int i = 0; i < p; ++i, ++r) {
            rm.tok[r] = st.pend_tok[b * D + i];
            rm.pos[r] = c + i; rm.seq[r] = b; rm.kind[r] = -1; rm.lim[r] = c + i + 1;
            rm.stg[r] = -1; rm.smask[r] = 0; rm.stg2[r] = -1;
        }
        for (int j = 0; j < D; ++j, ++r) {
            rm.tok[r] = j == 0 ? st.last_tok[b] : mask_id;
            rm.pos[r] = n - 1 + j; rm.seq[r] = b; rm.kind[r] = j; rm.lim[r] = n - 1;
            rm.stg[r] = stg0 + b; rm.smask[r] = (1 << (causal ? j + 1 : D)) - 1;   // block keys: all D, or (causal variant) up to the row itself
            rm.stg2[r] = -1;
            rm.blk_row[b * D + j] = r;
        }
        int rows = p + D, g = grp0[b];
        for (int o = 0; o < rows; o += gr, ++g) {
            const int gn = min(gr, rows - o);
            rm.grp_row0[g] = row0[b] + o;
            rm.grp_n[g] = gn;
            rm.grp_seq[g] = b;
            rm.grp_stg[g] = stg0 + b;
            rm.grp_stg2[g] = -1;
            // largest visible-key limit of the group's rows: pending row i has c + i + 1, block rows n - 1
            const int last = o + gn - 1, lim_max = o < p ? c + min(last, p - 1) + 1 : n - 1;
            rm.grp_hint[g] = attn_group_hint(lim_max, gn, cp_s);
        }
    }
    if (!E) return;
    __syncthreads();   // the rows' tokens are written by this workgroup
    embed_rows(x, E, rm.tok, row0[B], h, V);
}

// Up to 8192 values (h = 1536, 8 rows, 12288: no difference to the launch of its own).
bool assemble_embeds(int B, int D, int h) { return B <= 4 && (long)B * 2 * D * h <= 8192; }

void launch_assemble_decode(hipStream_t s, const SeqState &st, const RowMeta &rm, int B, int D, int mask_id, int group_rows, int staging_base,
                            int causal, int n_kv_heads, int chunk_floor, int dtype, float *x, const void *E, int h, int V)
{
    if (dtype == 0) hipLaunchKernelGGL(assemble_decode_k<float>, dim3(1), dim3(256), 0, s, st, rm, B, D, mask_id, group_rows, staging_base, causal, n_kv_heads, chunk_floor, x, (const float *)E, h, V);
    else hipLaunchKernelGGL(assemble_decode_k<bf16_t>, dim3(1), dim3(256), 0, s, st, rm, B, D, mask_id, group_rows, staging_base, causal, n_kv_heads, chunk_floor, x, (const bf16_t *)E, h, V);
}

// Rows of the verification pass of a self-speculative step (Sec. 3.4, "Self-Speculative Decoding").  With yhat^1..yhat^D
// the tokens of the step just computed and n the number of known tokens, verification input j (j = 2..D; input 1 is
// the step itself) is the sequence extended by yhat^1..yhat^{j-1}:
//   j-2 causal rows   yhat^1..yhat^{j-2} at positions n..n+j-3
//   D block rows      [yhat^{j-1}, [m] x (D-1)] at positions n+j-2 ..
// All of them see the cache keys [0, n) (written by the step: every known token including x_last has its causal K/V
// there) and keep their own K/V in staging tiles; nothing is written to the cache.  The causal row of yhat^i is the
// same in every input that has it (same token, same position, same visible keys), so it is computed once per sequence:
// a sequence contributes its D-2 causal rows, then the D block rows of each input, (D-2) + (D-1) D rows in all.  Only the
// first block row of each input goes through the LM head: its arg-max is ytilde^j.
//   shared != 0 (all those rows fit the 16 slots of one tile, D <= 4): one tile per sequence; the causal rows sit in slots
//     0 .. D-3, input j's block in slots D-2 + (j-2) D ..., and its rows see the causal slots 0 .. j-3 and their own block.
//     The rows of a sequence then form row groups regardless of the input they belong to.
//   shared == 0: the causal rows live in a tile of their own (the sequence's last staging tile), every input's block in the
//     input's tile; a block row reads two staging tiles, its input's (slots 0 .. D-1) and the causal one (slots 0 .. j-3,
//     upper half of its slot mask).  Row groups do not straddle inputs, so a group reads at most these two tiles.
__global__ void assemble_verify_k(SeqState st, RowMeta rm, int B, int D, int mask_id, int gr, int stg0, int causal, int shared, int Hkv, int cp_floor)
{
    __shared__ int row0[1025], grp0[1025], cp_s;
    const int rows_seq = (D - 2) + (D - 1) * D;
    const int groups_seq = verify_groups_per_seq(D, gr);
    if (threadIdx.x == 0) {
        long tiles = 0;
        for (int b = 0; b < B; ++b) {
            row0[b] = b * rows_seq; grp0[b] = b * groups_seq;
            tiles += (long)groups_seq * ((st.n[b] + PAGE - 1) / PAGE);
        }
        rm.counts[0] = B * rows_seq; rm.counts[1] = B * groups_seq; rm.counts[2] = B * (D - 1);
        cp_s = attn_chunk_pages(tiles * Hkv, cp_floor);
        rm.counts[3] = cp_s;
    }
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += blockDim.x) {
        const int n = st.n[b];
        const int32_t *yhat = st.last_ids + b * D;
        int r = row0[b], g = grp0[b];
        if (shared) {
            const int tile = stg0 + B + b * D;
            for (int i = 0; i < D - 2; ++i, ++r) {
                rm.tok[r] = yhat[i]; rm.pos[r] = n + i; rm.seq[r] = b; rm.kind[r] = i; rm.lim[r] = n;
                rm.stg[r] = tile; rm.smask[r] = (1 << (i + 1)) - 1; rm.stg2[r] = -1;
            }
            for (int j = 2; j <= D; ++j) {
                const int base = (D - 2) + (j - 2) * D, common = (1 << (j - 2)) - 1;
                for (int t = 0; t < D; ++t, ++r) {
                    rm.tok[r] = t == 0 ? yhat[j - 2] : mask_id; rm.pos[r] = n + j - 2 + t; rm.seq[r] = b; rm.kind[r] = base + t;
                    rm.lim[r] = n; rm.stg[r] = tile; rm.smask[r] = common | (((1 << (causal ? t + 1 : D)) - 1) << base); rm.stg2[r] = -1;
                    if (t == 0) rm.blk_row[b * (D - 1) + (j - 2)] = r;
                }
            }
            for (int o = 0; o < rows_seq; o += gr, ++g) {
                rm.grp_row0[g] = row0[b] + o;
                rm.grp_n[g] = min(gr, rows_seq - o);
                rm.grp_seq[g] = b;
                rm.grp_stg[g] = tile; rm.grp_stg2[g] = -1;
                rm.grp_hint[g] = attn_group_hint(n, min(gr, rows_seq - o), cp_s);
            }
            continue;
        }
        // tiles of sequence b: stg0 + B + b D + (j - 2) for input j, and stg0 + B + b D + (D - 1) for the causal rows
        const int ctile = stg0 + B + b * D + (D - 1);
        for (int i = 0; i < D - 2; ++i, ++r) {
            rm.tok[r] = yhat[i]; rm.pos[r] = n + i; rm.seq[r] = b; rm.kind[r] = i; rm.lim[r] = n;
            rm.stg[r] = ctile; rm.smask[r] = (1 << (i + 1)) - 1; rm.stg2[r] = -1;
        }
        for (int o = 0; o < D - 2; o += gr, ++g) {
            rm.grp_row0[g] = row0[b] + o;
            rm.grp_n[g] = min(gr, D - 2 - o);
            rm.grp_seq[g] = b;
            rm.grp_stg[g] = ctile; rm.grp_stg2[g] = -1;
            rm.grp_hint[g] = attn_group_hint(n, min(gr, D - 2 - o), cp_s);
        }
        for (int j = 2; j <= D; ++j) {
            const int tile = stg0 + B + b * D + (j - 2), first = r;
            const int common = (1 << (j - 2)) - 1;   // causal slots 0 .. j-3 of the causal tile
            for (int t = 0; t < D; ++t, ++r) {
                rm.tok[r] = t == 0 ? yhat[j - 2] : mask_id; rm.pos[r] = n + j - 2 + t; rm.seq[r] = b; rm.kind[r] = t;
                rm.lim[r] = n; rm.stg[r] = tile; rm.stg2[r] = common ? ctile : -1;
                rm.smask[r] = (int32_t)((uint32_t)((1 << (causal ? t + 1 : D)) - 1) | ((uint32_t)common << 16));
                if (t == 0) rm.blk_row[b * (D - 1) + (j - 2)] = r;
            }
            for (int o = 0; o < D; o += gr, ++g) {
                rm.grp_row0[g] = first + o;
                rm.grp_n[g] = min(gr, D - o);
                rm.grp_seq[g] = b;
                rm.grp_stg[g] = tile; rm.grp_stg2[g] = common ? ctile : -1;
                rm.grp_hint[g] = attn_group_hint(n, min(gr, D - o), cp_s);
            }
        }
    }
}

int verify_rows_per_seq(int D, bool *shared_tile)
{
    if (D < 2) { if (shared_tile) *shared_tile = true; return 0; }
    if (shared_tile) *shared_tile = (D - 2) + (D - 1) * D <= PAGE;   // every row of a sequence fits one staging tile
    return (D - 2) + (D - 1) * D;
}

void launch_assemble_verify(hipStream_t s, const SeqState &st, const RowMeta &rm, int B, int D, int mask_id, int group_rows,
                            int staging_base, int causal, int n_kv_heads, int chunk_floor)
{
    bool shared;
    verify_rows_per_seq(D, &shared);
    hipLaunchKernelGGL(assemble_verify_k, dim3(1), dim3(256), 0, s, st, rm, B, D, mask_id, group_rows, staging_base, causal, shared ? 1 : 0, n_kv_heads,
                       chunk_floor);
}

// gamma_verify (Eq. 10) from the step's tokens yhat and the verification predictions (ids_rows: ytilde^2..ytilde^D per
// sequence; ytilde^1 = yhat^1 because input 1 is the step itself).  rule 0: longest prefix on which all positions
// agree; rule 1: the largest agreeing index, as the equation is printed.  The result replaces the step's own count,
// so that a commit without overrides publishes the verified tokens.
__global__ void verify_accept_k(SeqState st, const int32_t *ids_rows, int B, int D, int rule, int32_t *ids_out, int32_t *count_out)
{
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int32_t *yhat = st.last_ids + b * D;
    int best = 1;
    bool run = true;
    for (int j = 1; j <= D; ++j) {
        int yt = j == 1 ? yhat[0] : ids_rows[b * (D - 1) + (j - 2)];
        if (ids_out) ids_out[b * D + j - 1] = yt;
        bool eq = yt == yhat[j - 1];
        run = run && eq;
        if (rule == 1 ? eq : run) best = j;
    }
    st.last_count[b] = best;
    if (count_out) count_out[b] = best;
}

void launch_verify_accept(hipStream_t s, const SeqState &st, const int32_t *ids_rows, int B, int D, int rule,
                          int32_t *ids_out, int32_t *count_out)
{
    hipLaunchKernelGGL(verify_accept_k, dim3((B + 63) / 64), dim3(64), 0, s, st, ids_rows, B, D, rule, ids_out, count_out);
}

// ------------------------------------------------------------------------------------------------ embedding
template <typename T>
__global__ void embed_k(float *x, const T *E, const int32_t *tok, const int32_t *pR, int h, int V)
{
    int r = blockIdx.x;
    if (r >= *pR) return;
    const T *e = E + (size_t)min(max(tok[r], 0), V - 1) * h;
    for (int k = threadIdx.x; k < h; k += blockDim.x) x[(size_t)r * h + k] = to_f<T>(e[k]);
}

void launch_embed(hipStream_t s, int dtype, float *x, const void *E, const RowMeta &rm, int max_rows, int h, int V)
{
    if (dtype == 0) hipLaunchKernelGGL(embed_k<float>, dim3(max_rows), dim3(256), 0, s, x, (const float *)E, rm.tok, rm.counts, h, V);
    else hipLaunchKernelGGL(embed_k<bf16_t>, dim3(max_rows), dim3(256), 0, s, x, (const bf16_t *)E, rm.tok, rm.counts, h, V);
}

// ------------------------------------------------------------------------------------------------ RMSNorm
__device__ inline float block_sum(float v, float *red)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    float t = 0.f;
    for (int i = 0; i < nw; ++i) t += red[i];
    return t;
}

// out[j,:] = x[row,:] * g / sqrt(mean(x[row,:]^2) + eps), row = row_index ? row_index[j] : j.  When the projection
// that produced the residual update was split along k, its partial sums (n_slabs slabs of [rows, h]) are first added
// to x[row,:] in slab order and written back, so the residual stream is complete after this kernel.
// A row lives in registers between the two passes (TH threads, NV float4 each, h <= 4 TH NV).
// Bound, with few rows: the memory round trips, one for the row and one per SU slabs; a row therefore gets the threads that let
// its slabs be requested together.  256 threads -> now: h = 5120, 8 rows 11.0 -> 6.5 us; h = 3584, 70 rows 7.8 -> 5.7 us, 512 rows
// 9.8 -> 8.6 us; h = 2048, 256 rows 6.5 -> 5.8 us.  With more rows than workgroups fit the chip at once: bandwidth, and small workgroups hide
// one row's reduction behind another's loads (see rmsnorm_t).
template <typename T, int TH, int NV, bool ORDERED>
__global__ __launch_bounds__(TH) void rmsnorm_k(T *out, float *x, const T *g, int h, float eps, const int32_t *row_index,
                                                const int32_t *p_count, int sure, const float *slabs, int n_slabs, size_t slab_stride)
{
    __shared__ float red[TH / 64];
    const int j = blockIdx.x;
    if (j >= sure && j >= *p_count) return;   // the first `sure` rows exist for certain: no wait for the device count
    const int row = row_index ? row_index[j] : j;
    float *xr = x + (size_t)row * h;
    float4 v[NV], gv[NV];   // the gains are requested together with the row, not after the reduction
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int k = (i * TH + threadIdx.x) * 4;
        v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        gv[i] = v[i];
        if (k < h) {
            v[i] = *(const float4 *)(xr + k);
            if constexpr (sizeof(T) == 2) {
                const uint2 u = *(const uint2 *)(g + k);
                gv[i] = make_float4(bf16_to_f((bf16_t)(u.x & 0xffff)), bf16_to_f((bf16_t)(u.x >> 16)),
                                    bf16_to_f((bf16_t)(u.y & 0xffff)), bf16_to_f((bf16_t)(u.y >> 16)));
            } else {
                gv[i] = *(const float4 *)(g + k);
            }
        }
    }
    // The slabs are added in slab order, but requested SU at a time (as many as the registers of the row width allow): one
    // memory round trip per SU slabs instead of one per slab.  Slabs past the end are neither requested nor added.
    constexpr int SU = NV <= 2 ? 8 : (NV <= 4 ? 4 : (NV == 8 ? 2 : 1));
    for (int s0 = 0; s0 < n_slabs; s0 += SU) {
        float4 p[SU][NV];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            if (s0 + u < n_slabs) {
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const int k = (i * TH + threadIdx.x) * 4;
                    p[u][i] = k < h ? *(const float4 *)(slabs + (s0 + u) * slab_stride + (size_t)row * h + k) : make_float4(0.f, 0.f, 0.f, 0.f);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            if (s0 + u < n_slabs) {
#pragma unroll
                for (int i = 0; i < NV; ++i) { v[i].x += p[u][i].x; v[i].y += p[u][i].y; v[i].z += p[u][i].z; v[i].w += p[u][i].w; }
            }
        }
    }
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int k = (i * TH + threadIdx.x) * 4;
        if (k < h && n_slabs > 0) *(float4 *)(xr + k) = v[i];
        ss += v[i].x * v[i].x + v[i].y * v[i].y + v[i].z * v[i].z + v[i].w * v[i].w;
    }
    ss = block_sum(ss, red);
    const float inv = 1.0f / sqrtf(ss / (float)h + eps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int k = (i * TH + threadIdx.x) * 4;
        if (k >= h) continue;
        const float o0 = v[i].x * inv * gv[i].x, o1 = v[i].y * inv * gv[i].y;
        const float o2 = v[i].z * inv * gv[i].z, o3 = v[i].w * inv * gv[i].w;
        T *dst = out + (ORDERED ? ordered_off(j, k, h) : (size_t)j * h + k);
        if constexpr (sizeof(T) == 2) {
            *(uint2 *)dst = make_uint2((uint32_t)f_to_bf16(o0) | ((uint32_t)f_to_bf16(o1) << 16),
                                       (uint32_t)f_to_bf16(o2) | ((uint32_t)f_to_bf16(o3) << 16));
        } else {
            *(float4 *)dst = make_float4(o0, o1, o2, o3);
        }
    }
}

template <typename T, bool ORDERED>
static void rmsnorm_t(hipStream_t s, void *out, float *x, const void *g, int h, float eps, const int32_t *row_index,
                      const int32_t *p_count, int max_rows, int min_rows, const float *slabs, int n_slabs, size_t slab_stride)
{
#define SDLM_RMS(TH, NV) hipLaunchKernelGGL((rmsnorm_k<T, TH, NV, ORDERED>), dim3(max_rows), dim3(TH), 0, s, (T *)out, x, (const T *)g, h, eps, row_index, p_count, min_rows, slabs, n_slabs, slab_stride)
    // Wide workgroups while those of all rows are on the chip at once (four a compute unit of 512 threads, two of 1024, one of 1024 with more
    // than 4096 values a row, for their registers), counted in certain rows: a step has few more, as a rule.  us, 256 threads / wide:
    //   h = 2048   1024 rows without slabs 4.4 / 4.4, 2048 rows 6.6 / 6.7
    //   h = 3584   512 rows, 4 slabs 9.3 / 8.4, without 4.5 / 4.4;  640 rows, 4 slabs 11.6 / 11.8, without 4.9 / 5.7;  4096 rows 18.2 / 20.8
    //   h = 5120   256 rows, 4 slabs 8.1 / 5.9, without 4.8 / 4.0;  384 rows, 4 slabs 11.1 / 11.1, without 5.0 / 5.9;  640 rows 15.4 / 18.1, 5.8 / 8.0
    const int rows = min_rows > 0 ? min(min_rows, max_rows) : max_rows;
    if (h <= 1024) SDLM_RMS(256, 1);
    else if (h <= 2048) { if (rows <= 1024) SDLM_RMS(512, 1); else SDLM_RMS(256, 2); }
    else if (h <= 4096) { if (rows <= 512) SDLM_RMS(1024, 1); else SDLM_RMS(256, 4); }
    else if (h <= 8192) { if (rows <= 256) SDLM_RMS(1024, 2); else SDLM_RMS(256, 8); }
    else { if (rows <= 256) SDLM_RMS(1024, 4); else SDLM_RMS(256, 16); }
#undef SDLM_RMS
}

void launch_rmsnorm(hipStream_t s, int dtype, void *out, float *x, const void *g, int h, float eps, const int32_t *row_index,
                    const int32_t *p_count, int max_rows, int min_rows, const float *slabs, int n_slabs, size_t slab_stride, bool ordered)
{
    // (the order as a template argument: as a run-time one it cost every norm 0.2 us)
    if (dtype == 0) rmsnorm_t<float, false>(s, out, x, g, h, eps, row_index, p_count, max_rows, min_rows, slabs, n_slabs, slab_stride);
    else if (ordered) rmsnorm_t<bf16_t, true>(s, out, x, g, h, eps, row_index, p_count, max_rows, min_rows, slabs, n_slabs, slab_stride);
    else rmsnorm_t<bf16_t, false>(s, out, x, g, h, eps, row_index, p_count, max_rows, min_rows, slabs, n_slabs, slab_stride);
}

// ------------------------------------------------------------------------------------------------ GEMM (FMA)
// Y[r, n] = sum_k X[r, k] * W[n, k]; 64x64 tile, 16-deep slices through LDS, 4x4 outputs per thread.
__device__ inline float silu_f(float v) { return v / (1.0f + __expf(-v)); }

template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_generic_k(GemmArgs a)
{
    const int R = min(*a.pR, a.max_rows);
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    if (m0 >= R) return;
    constexpr bool DUAL = EPI == EPI_SWIGLU;
    __shared__ float Xs[16][65], Ws[16][65], Us[DUAL ? 16 : 1][65];
    const T *X = (const T *)a.X, *W = (const T *)a.W, *W2 = (const T *)a.W2;
    const int t = threadIdx.x, tx = t & 15, ty = t >> 4, K = a.K, N = a.N;
    float acc[4][4] = {}, acc2[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += 16) {
        for (int e = t; e < 1024; e += 256) {
            int row = e >> 4, kk = e & 15;
            bool kin = k0 + kk < K;
            Xs[kk][row] = (kin && m0 + row < R) ? to_f<T>(X[(size_t)(m0 + row) * K + k0 + kk]) : 0.f;
            bool nin = kin && n0 + row < N;
            Ws[kk][row] = nin ? to_f<T>(W[(size_t)(n0 + row) * K + k0 + kk]) : 0.f;
            if (DUAL) Us[kk][row] = nin ? to_f<T>(W2[(size_t)(n0 + row) * K + k0 + kk]) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            float xv[4], wv[4], uv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { xv[i] = Xs[kk][ty * 4 + i]; wv[i] = Ws[kk][tx * 4 + i]; uv[i] = DUAL ? Us[kk][tx * 4 + i] : 0.f; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[i][j] += xv[i] * wv[j];
                    if (DUAL) acc2[i][j] += xv[i] * uv[j];
                }
        }
        __syncthreads();
    }
    for (int i = 0; i < 4; ++i) {
        int r = m0 + ty * 4 + i;
        if (r >= R) continue;
        for (int j = 0; j < 4; ++j) {
            int n = n0 + tx * 4 + j;
            if (n >= N) continue;
            size_t o = (size_t)r * N + n;
            if (EPI == EPI_STORE_F32) a.Yf[o] = acc[i][j] + (a.bias ? to_f<T>(((const T *)a.bias)[n]) : 0.f);
            else if (EPI == EPI_RESID) a.Yf[o] += acc[i][j];
            else if (EPI == EPI_SWIGLU) ((T *)a.Yt)[o] = from_f<T>(silu_f(acc[i][j]) * acc2[i][j]);
            else a.Yf[o] = acc[i][j] * a.scale;
        }
    }
}

// The same products without LDS, for few rows and for K whose rows are whole 16-byte groups (see gemm_generic_go).
// Sixteen lanes share an output column: each walks k in steps of 16 VE elements, and the sixteen partial sums are added by a
// fixed tree, so an output's sum does not depend on RT, CN or the other rows of the launch.  A few rows leave the 64x64
// tiles a handful of workgroups with a serial k loop and a barrier pair per 16 k (K = 688, N = 256: 4 workgroups, 68 us; here
// 16 workgroups whose loads are all requested at once, 5 us, which is the launch itself).  RT x CN outputs per lane group
// balance the loads per FMA: 8 x 1 spreads a small product over as many wavefronts as possible, 32 x 4 re-uses each loaded
// vector 8 times more often.
template <typename T> struct Vec16;   // 16 bytes of T as floats
template <> struct Vec16<float> {
    static constexpr int N = 4;
    float4 r;
    __device__ inline void load(const float *p) { r = *(const float4 *)p; }
    __device__ inline void zero() { r = make_float4(0.f, 0.f, 0.f, 0.f); }
    __device__ inline float at(int e) const { return e == 0 ? r.x : e == 1 ? r.y : e == 2 ? r.z : r.w; }
};
template <> struct Vec16<bf16_t> {
    static constexpr int N = 8;
    uint4 r;
    __device__ inline void load(const bf16_t *p) { r = *(const uint4 *)p; }
    __device__ inline void zero() { r = make_uint4(0, 0, 0, 0); }
    __device__ inline float at(int e) const
    {
        const uint32_t w = e < 2 ? r.x : e < 4 ? r.y : e < 6 ? r.z : r.w;
        return bf16_to_f((bf16_t)((e & 1) ? w >> 16 : w & 0xffffu));
    }
};

template <typename T, int EPI, int RT, int CN>
__global__ __launch_bounds__(256) void gemm_rows_k(GemmArgs a)
{
    const int R = min(*a.pR, a.max_rows);
    const int r0 = blockIdx.y * RT;
    if (r0 >= R) return;
    constexpr bool DUAL = EPI == EPI_SWIGLU;
    constexpr int VE = Vec16<T>::N, U = RT == 8 ? 4 : 1;   // vectors requested per round and operand row
    const T *X = (const T *)a.X, *W = (const T *)a.W, *W2 = (const T *)a.W2;
    const int lane = threadIdx.x & 63, l16 = lane & 15, K = a.K, N = a.N;
    const int n0 = (blockIdx.x * 16 + (threadIdx.x >> 6) * 4 + (lane >> 4)) * CN;
    const T *xp[RT], *wp[CN], *up[DUAL ? CN : 1];
#pragma unroll
    for (int i = 0; i < RT; ++i) xp[i] = X + (size_t)min(r0 + i, R - 1) * K;
#pragma unroll
    for (int c = 0; c < CN; ++c) {
        wp[c] = W + (size_t)min(n0 + c, N - 1) * K;
        if constexpr (DUAL) up[c] = W2 + (size_t)min(n0 + c, N - 1) * K;
    }
    float acc[CN][RT], acc2[DUAL ? CN : 1][RT];
#pragma unroll
    for (int c = 0; c < CN; ++c)
#pragma unroll
        for (int i = 0; i < RT; ++i) { acc[c][i] = 0.f; if constexpr (DUAL) acc2[c][i] = 0.f; }
    for (int k0 = l16 * VE; k0 < K; k0 += 16 * VE * U) {
        Vec16<T> w[U][CN], u2[U][DUAL ? CN : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * 16 * VE;
#pragma unroll
            for (int c = 0; c < CN; ++c) {
                w[u][c].zero();
                if (k < K) w[u][c].load(wp[c] + k);
                if constexpr (DUAL) { u2[u][c].zero(); if (k < K) u2[u][c].load(up[c] + k); }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * 16 * VE;
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                Vec16<T> x;
                x.zero();
                if (k < K) x.load(xp[i] + k);
#pragma unroll
                for (int c = 0; c < CN; ++c)
#pragma unroll
                    for (int e = 0; e < VE; ++e) {
                        acc[c][i] = fmaf(x.at(e), w[u][c].at(e), acc[c][i]);
                        if constexpr (DUAL) acc2[c][i] = fmaf(x.at(e), u2[u][c].at(e), acc2[c][i]);
                    }
            }
        }
    }
    // sum over the sixteen lanes, halving the rows a lane carries with the distance (8, 4, 2), then the last pair
    auto reduce8 = [&](float (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float keep = (l16 & 8) ? v[i + 4] : v[i], send = (l16 & 8) ? v[i] : v[i + 4];
            v[i] = keep + __shfl_xor(send, 8);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float keep = (l16 & 4) ? v[i + 2] : v[i], send = (l16 & 4) ? v[i] : v[i + 2];
            v[i] = keep + __shfl_xor(send, 4);
        }
        const float keep = (l16 & 2) ? v[1] : v[0], send = (l16 & 2) ? v[0] : v[1];
        v[0] = keep + __shfl_xor(send, 2);
        v[0] += __shfl_xor(v[0], 1);
        return v[0];
    };
    const int rsub = ((l16 >> 3) & 1) * 4 + ((l16 >> 2) & 1) * 2 + ((l16 >> 1) & 1);
#pragma unroll
    for (int c = 0; c < CN; ++c)
#pragma unroll
        for (int b = 0; b < RT; b += 8) {
            float v[8], v2[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) { v[i] = acc[c][b + i]; v2[i] = DUAL ? acc2[DUAL ? c : 0][b + i] : 0.f; }
            const float s = reduce8(v);
            float s2 = 0.f;
            if constexpr (DUAL) s2 = reduce8(v2);
            const int r = r0 + b + rsub, n = n0 + c;
            if ((l16 & 1) || r >= R || n >= N) continue;
            const size_t o = (size_t)r * N + n;
            if (EPI == EPI_STORE_F32) a.Yf[o] = s + (a.bias ? to_f<T>(((const T *)a.bias)[n]) : 0.f);
            else if (EPI == EPI_RESID) a.Yf[o] += s;
            else if (EPI == EPI_SWIGLU) ((T *)a.Yt)[o] = from_f<T>(silu_f(s) * s2);
            else a.Yf[o] = s * a.scale;
        }
}

// ------------------------------------------------------------------------------------------------ steps of few rows
// A step of a small model on this path is a chain of launches with next to nothing in them (2.4 us each at the least), so the norms,
// the rotation and the K/V placement join the products they feed.  A product of at most FEW_ROWS rows reads the residual stream itself: the
// lanes that walk a column's k also sum the squares of the rows, and the row's factor 1 / rms is applied to the finished sum.
// A wavefront owns a column and walks k with all of its lanes, eight rows at a time; four columns a workgroup, and workgroups of neighbouring columns on one
// XCD, so that a cache line of results has one owner (N = 256, K = 256, eight XCDs in every line of the residual stream: 6.9 us, so 2.9).  Sixteen lanes
// a column request the rows four times over and walk k in turns (K = 688: 7.3 us, so 5.3); four columns a wavefront take longer with their arithmetic (8.0).
// us a step, norms and products apart -> now: h = 256, F = 688, 2 layers, 8 rows 84.7 -> 60.1; h = 896, F = 4864, 4 layers fp32 8 / 16 / 32 rows 417 -> 258 / 438 -> 308 / 470 -> 370,
// bf16 307 -> 219 / 330 -> 272 / 352 -> 340; h = 2048, F = 11008, 2 layers fp32 477 -> 350 / 551 -> 482 / 738 -> 674.  The requests of the rows, fp32 and repeated for
// every column and group of eight rows, grow with the layer, what they save does not: the line is generic_few_pays.
constexpr int FEW_ROWS = 32;

struct FewArgs {
    const void *X;                  // [R, K]: fp32 residual stream (NORM) or activations of the storage type
    const void *gain;               // [K], NORM
    const int32_t *row_index;       // NORM: row of X behind each row of the product, null: the same
    const void *W, *W2, *bias;
    float *Yf;
    void *Yt;
    const int32_t *pR;
    int max_rows, N, K;
    float scale, eps;
};

// Vec16<T>::N consecutive elements of a row of X as floats.
template <typename T, bool NORM> struct FewX {
    Vec16<T> v;
    __device__ inline void load(const void *p, size_t o) { v.load((const T *)p + o); }
    __device__ inline float at(int e) const { return v.at(e); }
};
template <> struct FewX<bf16_t, true> {
    Vec16<float> a, b;
    __device__ inline void load(const void *p, size_t o) { a.load((const float *)p + o); b.load((const float *)p + o + 4); }
    __device__ inline float at(int e) const { return e < 4 ? a.at(e) : b.at(e - 4); }
};

// Sums of eight values over the wavefront, by a fixed tree: the values a lane carries halve while there are several, so that lane l ends with
// the sum of value l / 8.
__device__ inline float few_sum(float (&v)[8], int lane)
{
#pragma unroll
    for (int h = 4, d = 32; h > 0; h >>= 1, d >>= 1)
#pragma unroll
        for (int i = 0; i < h; ++i) {
            const float keep = (lane & d) ? v[i + h] : v[i], send = (lane & d) ? v[i] : v[i + h];
            v[i] = keep + __shfl_xor(send, d);
        }
#pragma unroll
    for (int d = 4; d > 0; d >>= 1) v[0] += __shfl_xor(v[0], d);
    return v[0];
}

// Products of NW weight rows with eight rows from r0 on; s[j] in lane l is the sum of w[j] and row r0 + l / 8.
template <typename T, bool NORM, int NW>
__device__ inline void few_dot(const FewArgs &a, const T *const (&w)[NW], int r0, int R, int lane, float (&s)[NW])
{
    constexpr int VE = Vec16<T>::N, U = NORM ? 2 : 3;   // k steps requested together, weights and rows
    const int K = a.K;
    size_t xo[8];
    float acc[NW][8], ss[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = min(r0 + i, R - 1);
        xo[i] = (size_t)(NORM && a.row_index ? a.row_index[r] : r) * K;
        ss[i] = 0.f;
#pragma unroll
        for (int j = 0; j < NW; ++j) acc[j][i] = 0.f;
    }
    for (int k0 = lane * VE; k0 < K; k0 += 64 * VE * U) {
        Vec16<T> wv[U][NW], gv[U];
        FewX<T, NORM> x[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u > 0 && k0 - lane * VE + u * 64 * VE >= K) break;   // no lane has such a step
            const int k = min(k0 + u * 64 * VE, K - VE);             // a lane beyond the end requests but does not use
#pragma unroll
            for (int j = 0; j < NW; ++j) wv[u][j].load(w[j] + k);
            if constexpr (NORM) gv[u].load((const T *)a.gain + k);
#pragma unroll
            for (int i = 0; i < 8; ++i) x[u][i].load(a.X, xo[i] + k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k0 + u * 64 * VE >= K) continue;
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int e = 0; e < VE; ++e) {
                    const float xe = x[u][i].at(e);
                    float xg = xe;
                    if constexpr (NORM) { ss[i] = fmaf(xe, xe, ss[i]); xg = xe * gv[u].at(e); }
#pragma unroll
                    for (int j = 0; j < NW; ++j) acc[j][i] = fmaf(xg, wv[u][j].at(e), acc[j][i]);
                }
        }
    }
    float inv = 1.f;
    if constexpr (NORM) inv = 1.0f / sqrtf(few_sum(ss, lane) / (float)K + a.eps);
#pragma unroll
    for (int j = 0; j < NW; ++j) s[j] = few_sum(acc[j], lane) * inv;
}

// Column of this wavefront: the workgroups of one XCD (blockIdx.x % 8) own neighbouring columns.
__device__ inline int few_column() { return ((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * 4 + (threadIdx.x >> 6); }

template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_few_k(FewArgs a)
{
    const int R = min(*a.pR, a.max_rows), r0 = blockIdx.y * 8, n = few_column();
    if (r0 >= R || n >= a.N) return;
    constexpr int NW = EPI == EPI_SWIGLU ? 2 : 1;
    const int lane = threadIdx.x & 63, r = r0 + (lane >> 3);
    const size_t o = (size_t)r * a.N + n;
    const bool mine = !(lane & 7) && r < R;
    float s[NW], old = 0.f;
    if (EPI == EPI_RESID && mine) old = a.Yf[o];   // requested with the operands
    const T *w[NW];
    w[0] = (const T *)a.W + (size_t)n * a.K;
    if constexpr (NW == 2) w[1] = (const T *)a.W2 + (size_t)n * a.K;
    few_dot<T, EPI != EPI_RESID, NW>(a, w, r0, R, lane, s);
    if (!mine) return;
    if (EPI == EPI_RESID) a.Yf[o] = old + s[0];
    else if (EPI == EPI_SWIGLU) ((T *)a.Yt)[o] = from_f<T>(silu_f(s[0]) * s[NW - 1]);
    else a.Yf[o] = s[0] * a.scale;
}

// QKV projection with the norm in front and rotation and K/V placement behind it (rope_scatter_k's): a wavefront owns a rotate-half pair.
template <typename T>
__global__ __launch_bounds__(256) void qkv_few_k(FewArgs a, T *q_out, T *pool, KvGeom kg, RowMeta rm, SeqState st, const float2 *rope, int Hq)
{
    const int R = min(*a.pR, a.max_rows), r0 = blockIdx.y * 8;
    const int d = kg.head_dim, half = d >> 1, Hk = kg.n_kv_heads, lane = threadIdx.x & 63, p = few_column(), head = p / half, i = p % half;
    if (r0 >= R || head >= Hq + 2 * Hk) return;
    const int r = r0 + (lane >> 3), rc = min(r, R - 1);
    const int pos = rm.pos[rc], kind = rm.kind[rc], b = rm.seq[rc], stg = rm.stg[rc];   // requested before the product
    const T *w[2] = {(const T *)a.W + (size_t)(head * d + i) * a.K, (const T *)a.W + (size_t)(head * d + i + half) * a.K};
    float x[2];
    few_dot<T, true, 2>(a, w, r0, R, lane, x);
    if ((lane & 7) || r >= R) return;
    if (a.bias) { x[0] += to_f<T>(((const T *)a.bias)[head * d + i]); x[1] += to_f<T>(((const T *)a.bias)[head * d + i + half]); }
    const bool is_v = head >= Hq + Hk;
    const float2 t = is_v ? make_float2(1.f, 0.f) : rope[(size_t)pos * half + i];
    const T lo = from_f<T>(is_v ? x[0] : x[0] * t.x - x[1] * t.y), hi = from_f<T>(is_v ? x[1] : x[1] * t.x + x[0] * t.y);
    if (head < Hq) {
        T *q = q_out + ((size_t)r * Hq + head) * d + i;
        q[0] = lo; q[half] = hi;
        return;
    }
    int page = stg, slot = kind;
    if (kind < 0) { page = st.page_table[(size_t)b * kg.pages_per_seq + pos / PAGE]; slot = pos % PAGE; }
    if (page < 0) return;   // unbacked position: only reachable after a reported pool exhaustion
    T *tile = pool + kg.tile(page, is_v ? head - Hq - Hk : head - Hq);
    if (!is_v) { tile[k_off(slot, i)] = lo; tile[k_off(slot, i + half)] = hi; }
    else { tile[PAGE * d + v_off(slot, i)] = lo; tile[PAGE * d + v_off(slot, i + half)] = hi; }
}

bool generic_few_applies(int dtype, int rows, int K) { return rows <= FEW_ROWS && K % (dtype == 0 ? 4 : 8) == 0; }

// Up to which layer, in 10^6 weights, for one to four groups of eight rows.  A layer of separate kernels against this one, us saved (negative: lost), over 170 random shapes:
//   fp32  8 rows  159 M +25, 223 M +87, 287 M -16, 357 M +56;  16 rows  92 M +23, 124 M +11, 148 M +62, 157 M -5, 179 M -16, 199 M -64;
//         24 rows  64 M +13, 71 M +33, 84 M +7, 88 M -7, 108 M -30, 140 M -40;  32 rows  36 M +35, 44 M +21, 52 M -3, 60 M -7 and +21, 83 M -19
//   bf16  8 rows  109 M +3, 125 M +2, 144 M +4, 173 M -13, 191 M -20, 232 M -28;  16 rows  31 M +10, 40 M +8, 45 M +3, 49 M +1, 60 M -5, 74 M -28, 165 M -61;
//         24 rows  12 M +6, 16 M +3, 19 M -5 and +4, 22 M 0, 27 M -5, 35 M -10;  32 rows  4.7 M +3, 8.3 M +3, 8.7 M -1, 10.6 M -2, 13.5 M -3
bool generic_few_pays(int dtype, int likely, double layer_elems)
{
    static const int fp32[4] = {360, 150, 80, 50}, bf16[4] = {160, 45, 18, 9};
    return likely <= FEW_ROWS && layer_elems <= 1e6 * (dtype == 0 ? fp32 : bf16)[(likely + 7) / 8 - 1];
}

// LM heads with the norm inside: up to 5000 (fp32) or 3000 (bf16) columns per group of eight rows; a wavefront a column, where the separate product has four columns a
// wavefront, outweighs the norm's launch beyond.  us a step saved, 160 shapes of h = 64 to 2048:
//   fp32  8 rows  V = 1500 +0.5 to +7, 4096 0 to +4, 6000 -1.4 to +4.5, 16000 -4;  16 rows  1500 0 to +6.5, 4096 -2.3 to +0.4, 8192 -3;  32 rows  512 +2, 1500 -2 to +6, 4096 -2
//   bf16  8 rows  V = 1500 +1.5 to +2.7, 4096 -0.7 to +2, 6000 -2;  16 rows  1500 +0.6 to +1.3, 4096 -3.4 to -5;  32 rows  512 +4 to +5.5, 1500 -2 to 0, 4096 -7 to -16
bool generic_few_head_pays(int dtype, int rows, int V) { return (long)V * ((rows + 7) / 8) <= (dtype == 0 ? 5000 : 3000); }

static dim3 few_grid(int cols, int rows) { return dim3((cols + 31) / 32 * 8, (rows + 7) / 8); }   // four columns a workgroup, a multiple of eight workgroups

template <typename T>
static void gemm_few_t(hipStream_t s, int epi, const FewArgs &a)
{
    const dim3 grid = few_grid(a.N, a.max_rows), block(256);
    if (epi == EPI_RESID) hipLaunchKernelGGL((gemm_few_k<T, EPI_RESID>), grid, block, 0, s, a);
    else if (epi == EPI_SWIGLU) hipLaunchKernelGGL((gemm_few_k<T, EPI_SWIGLU>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((gemm_few_k<T, EPI_LOGITS>), grid, block, 0, s, a);
}

// Residual: X is the input of the projection.  Gate/up and logits: X is the residual stream, normalised here.
void launch_gemm_few(hipStream_t s, int dtype, int epi, const GemmArgs &g, const void *gain, float eps, const int32_t *row_index)
{
    const FewArgs a{g.X, gain, row_index, g.W, g.W2, nullptr, g.Yf, g.Yt, g.pR, g.max_rows, g.N, g.K, g.scale, eps};
    if (dtype == 0) gemm_few_t<float>(s, epi, a);
    else gemm_few_t<bf16_t>(s, epi, a);
}

template <typename T>
static void qkv_few_t(hipStream_t s, const FewArgs &a, void *q_out, void *pool_layer, const KvGeom &kg, const RowMeta &rm, const SeqState &st, const float2 *rope, int Hq)
{
    const int pairs = (Hq + 2 * kg.n_kv_heads) * kg.head_dim / 2;
    hipLaunchKernelGGL((qkv_few_k<T>), few_grid(pairs, a.max_rows), dim3(256), 0, s, a, (T *)q_out, (T *)pool_layer, kg, rm, st, rope, Hq);
}

void launch_qkv_few(hipStream_t s, int dtype, const GemmArgs &g, const void *gain, float eps, void *q_out, void *pool_layer, const KvGeom &kg, const RowMeta &rm,
                    const SeqState &st, const float2 *rope, int n_q_heads)
{
    const FewArgs a{g.X, gain, nullptr, g.W, nullptr, g.bias, nullptr, nullptr, g.pR, g.max_rows, g.N, g.K, 1.f, eps};
    if (dtype == 0) qkv_few_t<float>(s, a, q_out, pool_layer, kg, rm, st, rope, n_q_heads);
    else qkv_few_t<bf16_t>(s, a, q_out, pool_layer, kg, rm, st, rope, n_q_heads);
}

// Which kernel: rows without LDS spend their time per output, tiles per 64 x 64 tile and k slice with little more until every
// compute unit has one or two.  `tiles` (N * rows / 4096) is where the lines lie, measured for both types, K from 128 to 8960 and N from 256
// to 151936 (us, rows without LDS -> tiles):
//   bf16  N = 896, K = 896: 1024 rows 86 -> 128, 2048 rows 172 -> 164, 4096 rows 331 -> 195;  K = 4864: 1024 rows 340 -> 774, 4096 1324 -> 1000
//   gate/up, N = 4864, K = 896: bf16 256 rows 139 -> 179, 384 rows 208 -> 190, 4096 rows 2138 -> 1233;  fp32 256 rows 191 -> 222, 384 rows 282 -> 233
//   short K (the lanes' final sum weighs more): gate/up, N = 3072, K = 128: bf16 96 rows 18.6 -> 24.5, 256 rows 41.7 -> 24.5
//   V = 151936, K = 896: fp32 16 rows 352 -> 437, 24 rows 523 -> 453; bf16 24 rows 350 -> 425, 32 rows 465 -> 430 (a tile's 64 rows are then
//   mostly padding, so the line is one of rows)
// 32-row groups of four columns serve the fp32 products of one matrix between one and one and a half tiles per unit, three of their
// workgroups a unit (N = 4096, K = 896: 384 rows 78 us, tiles 135, eight-row groups 172; 448 rows 181, tiles 137).  They lose
// with bf16 (384 rows 102, and 245 for gate/up, N = 4864, against 208) and with two matrices.
template <typename T, int EPI>
static void gemm_generic_go(hipStream_t s, const GemmArgs &a)
{
    constexpr bool FP32 = sizeof(T) == 4, ONE32 = FP32 && EPI != EPI_SWIGLU;
    const long outputs = (long)a.N * a.max_rows;
    const bool many = a.max_rows > (FP32 ? 16 : 24) && outputs * 512 > (ONE32 ? 384L : 352L) * 4096 * min(a.K, 512);
    if (a.K % Vec16<T>::N != 0 || many) {
        hipLaunchKernelGGL((gemm_generic_k<T, EPI>), dim3((a.N + 63) / 64, (a.max_rows + 63) / 64), dim3(256), 0, s, a);
        return;
    }
    if constexpr (ONE32) {
        const dim3 wide((a.N + 63) / 64, (a.max_rows + 31) / 32);
        if (a.max_rows > 8 && (long)wide.x * wide.y >= 512) {
            hipLaunchKernelGGL((gemm_rows_k<T, EPI, 32, 4>), wide, dim3(256), 0, s, a);
            return;
        }
    }
    hipLaunchKernelGGL((gemm_rows_k<T, EPI, 8, 1>), dim3((a.N + 15) / 16, (a.max_rows + 7) / 8), dim3(256), 0, s, a);
}

template <typename T>
static void gemm_generic_t(hipStream_t s, int epi, const GemmArgs &a)
{
    switch (epi) {
    case EPI_STORE_F32: gemm_generic_go<T, EPI_STORE_F32>(s, a); break;
    case EPI_RESID: gemm_generic_go<T, EPI_RESID>(s, a); break;
    case EPI_SWIGLU: gemm_generic_go<T, EPI_SWIGLU>(s, a); break;
    default: gemm_generic_go<T, EPI_LOGITS>(s, a); break;
    }
}

void launch_gemm_generic(hipStream_t s, int dtype, int epi, const GemmArgs &a)
{
    if (dtype == 0) gemm_generic_t<float>(s, epi, a);
    else gemm_generic_t<bf16_t>(s, epi, a);
}

// ------------------------------------------------------------------------------------------------ RoPE + K/V placement
// qkv: raw projections [R, (Hq + 2 Hkv) d] fp32, given as n_slabs partial sums that are added in order.  Queries and keys are rotated at the row's position (rotate-half
// pairing i <-> i + d/2).  A pending row's K/V go to the cache slot of its position: they are final.  A block
// row's K/V (and, in a verification pass, every row's) go to slot `kind` of the row's staging tile: they are never cached.
// grid (rows, ceil((Hq + 2 Hkv) / 4)): one wavefront per (row, head), lane i < d/2 owns the pair (i, i + d/2).
template <typename T>
__global__ __launch_bounds__(256) void rope_scatter_k(const float *qkv, int n_slabs, size_t slab_stride, T *q_out, T *pool, KvGeom kg,
                                                      RowMeta rm, SeqState st, const float2 *rope, int Hq, int sure)
{
    const int r = blockIdx.x;
    const int d = kg.head_dim, half = d >> 1, Hk = kg.n_kv_heads, nq = Hq * d, nk = Hk * d;
    const int head = blockIdx.y * 4 + (threadIdx.x >> 6), i = threadIdx.x & 63;   // heads: Hq of q, then Hkv of k, then Hkv of v
    if (head >= Hq + 2 * Hk || i >= half || (r >= sure && r >= rm.counts[0])) return;   // certain rows: no wait for the count
    const float *src = qkv + (size_t)r * (nq + 2 * nk) + head * d + i;
    const int pos = rm.pos[r], kind = rm.kind[r], b = rm.seq[r], stg = rm.stg[r];   // requested together with the projections
    float x0 = src[0], x1 = src[half];
    for (int s0 = 1; s0 < n_slabs; s0 += 4) {   // four slabs per memory round trip, added in slab order
        float p0[4], p1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t o = (size_t)min(s0 + u, n_slabs - 1) * slab_stride;
            p0[u] = src[o];
            p1[u] = src[o + half];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (s0 + u < n_slabs) { x0 += p0[u]; x1 += p1[u]; }
    }
    if (head < Hq) {
        const float2 t = rope[(size_t)pos * half + i];
        T *q = q_out + (size_t)r * nq + head * d + i;
        q[0] = from_f<T>(x0 * t.x - x1 * t.y);
        q[half] = from_f<T>(x1 * t.x + x0 * t.y);
        return;
    }
    int page, slot;
    if (kind < 0) { page = st.page_table[(size_t)b * kg.pages_per_seq + pos / PAGE]; slot = pos % PAGE; }
    else { page = stg; slot = kind; }
    if (page < 0) return;   // unbacked position: only reachable after a reported pool exhaustion
    const bool is_k = head < Hq + Hk;
    const int hk = is_k ? head - Hq : head - Hq - Hk;
    T *tile = pool + kg.tile(page, hk);
    if (is_k) {
        const float2 t = rope[(size_t)pos * half + i];
        tile[k_off(slot, i)] = from_f<T>(x0 * t.x - x1 * t.y);
        tile[k_off(slot, i + half)] = from_f<T>(x1 * t.x + x0 * t.y);
    } else {
        T *Vb = tile + PAGE * d;
        Vb[v_off(slot, i)] = from_f<T>(x0);
        Vb[v_off(slot, i + half)] = from_f<T>(x1);
    }
}

void launch_rope_scatter(hipStream_t s, int dtype, const float *qkv, int n_slabs, size_t slab_stride, void *q_out, void *pool_layer,
                         const KvGeom &kg, const RowMeta &rm, const SeqState &st, const float2 *rope, int n_q_heads, int max_rows, int min_rows)
{
    dim3 grid(max_rows, (n_q_heads + 2 * kg.n_kv_heads + 3) / 4);
    if (dtype == 0) hipLaunchKernelGGL(rope_scatter_k<float>, grid, dim3(256), 0, s, qkv, n_slabs, slab_stride, (float *)q_out, (float *)pool_layer, kg, rm, st, rope, n_q_heads, min_rows);
    else hipLaunchKernelGGL(rope_scatter_k<bf16_t>, grid, dim3(256), 0, s, qkv, n_slabs, slab_stride, (bf16_t *)q_out, (bf16_t *)pool_layer, kg, rm, st, rope, n_q_heads, min_rows);
}

// ------------------------------------------------------------------------------------------------ attention
// One workgroup per (row, query head).  Keys: the cache positions [0, lim) of the row's sequence and the slots of
// the row's staging tiles named by its slot masks; for a block row these are the D keys of its block (mask equation, Sec. 3.3:
// causal below the block start, full mutual attention inside the block).  They form a list of 16-key tiles (the cache's, then
// the staging tiles); the four wavefronts take four tiles at a time with a running (max, sum, output) each, merged at the end.
// Scores: one lane per key, the key's features as 16-byte loads.  Output: one lane per feature, four slots per load (the
// tile's own order), the weights handed over through LDS: one lane per key would read every value alone (20.7 us at 64 to 128
// keys and head_dim 64; this 5 us, the launch and three dependent memory round trips).
template <typename T, int HD>
__global__ __launch_bounds__(256) void attn_generic_k(const T *q, T *out, const T *pool, KvGeom kg, RowMeta rm, SeqState st,
                                                      int Hq)
{
    const int r = blockIdx.y;
    if (r >= rm.counts[0]) return;
    constexpr int FD = (HD + 63) / 64;   // features per lane
    const int hq = blockIdx.x, G = Hq / kg.n_kv_heads, hk = hq / G, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b = rm.seq[r], lim = rm.lim[r], stg = rm.stg[r], stg2 = rm.stg2[r];
    const uint32_t sm_all = (uint32_t)rm.smask[r];
    const uint32_t smask = stg >= 0 ? sm_all & 0xffffu : 0u, smask2 = stg2 >= 0 ? sm_all >> 16 : 0u;
    const int n_cache = (lim + PAGE - 1) / PAGE, at2 = smask2 ? n_cache : -1, at1 = smask ? n_cache + (smask2 ? 1 : 0) : -1;
    const int n_tiles = n_cache + (smask ? 1 : 0) + (smask2 ? 1 : 0);
    __shared__ float qs[HD];
    __shared__ __attribute__((aligned(16))) float ps[4][64];
    __shared__ float wm[4], wl[4], wo[4][HD];
    const float scale = 1.0f / sqrtf((float)HD);
    for (int i = threadIdx.x; i < HD; i += 256) qs[i] = to_f<T>(q[((size_t)r * Hq + hq) * HD + i]);
    __syncthreads();
    float m = -INFINITY, l = 0.f, o[FD];
#pragma unroll
    for (int f = 0; f < FD; ++f) o[f] = 0.f;
    for (int t0 = wave * 4; t0 < n_tiles; t0 += 16) {
        const int t = t0 + (lane >> 4), slot = lane & 15;
        int page = 0;
        bool vis = false;
        if (t == at1) { page = stg; vis = (smask >> slot) & 1u; }
        else if (t == at2) { page = stg2; vis = (smask2 >> slot) & 1u; }
        else if (t < n_cache) { page = max(st.page_table[(size_t)b * kg.pages_per_seq + t], 0); vis = t * PAGE + slot < lim; }
        float s = -INFINITY;
        if (vis) {
            const T *Kb = pool + kg.tile(page, hk) + slot * 8;
            float dot = 0.f;
            Vec16<T> kv[HD / Vec16<T>::N];
#pragma unroll
            for (int i = 0; i < HD / Vec16<T>::N; ++i) kv[i].load(Kb + k_off(0, i * Vec16<T>::N));
#pragma unroll
            for (int i = 0; i < HD / Vec16<T>::N; ++i)
#pragma unroll
                for (int e = 0; e < Vec16<T>::N; ++e) dot += qs[i * Vec16<T>::N + e] * kv[i].at(e);
            s = dot * scale;
        }
        float mx = s;
        for (int d = 32; d > 0; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
        const float mn = fmaxf(m, mx);
        const float corr = m == -INFINITY ? 0.f : __expf(m - mn), p = s == -INFINITY ? 0.f : __expf(s - mn);   // a NaN score stays one, whatever mn is
        m = mn;
        l = l * corr + p;
#pragma unroll
        for (int f = 0; f < FD; ++f) o[f] *= corr;
        ps[wave][lane] = p;   // read back by the same wavefront only
        __builtin_amdgcn_wave_barrier();
        // An unseen slot may hold anything, and 0 times a non-finite value is not 0: such values are cleared.
        auto add_values = [&](int tt, uint32_t seen_t, auto whole) {   // seen_t: the tile's slots that the row sees; whole: all of them
            const T *Vb = pool + kg.tile(__shfl(page, tt * 16), hk) + PAGE * HD;
#pragma unroll
            for (int f = 0; f < FD; ++f) {
                const int i = lane + f * 64;
                if (i >= HD) continue;
#pragma unroll
                for (int sg = 0; sg < 4; ++sg) {
                    const float4 p4 = *(const float4 *)&ps[wave][tt * 16 + sg * 4];
                    uint32_t v[4];
                    if constexpr (sizeof(T) == 4) {
                        const uint4 x = *(const uint4 *)(Vb + v_off(sg * 4, i));
                        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
                    } else {
                        const uint2 x = *(const uint2 *)(Vb + v_off(sg * 4, i));
                        v[0] = x.x << 16; v[1] = x.x & 0xffff0000u; v[2] = x.y << 16; v[3] = x.y & 0xffff0000u;
                    }
                    if constexpr (!whole) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] &= 0u - ((seen_t >> (sg * 4 + e)) & 1u);
                    }
                    o[f] += p4.x * __uint_as_float(v[0]) + p4.y * __uint_as_float(v[1]) + p4.z * __uint_as_float(v[2]) + p4.w * __uint_as_float(v[3]);
                }
            }
        };
        const uint64_t seen = __ballot(vis);   // bit 16 tt + slot: the row sees that slot of tile t0 + tt
        if (seen == ~0ull) {   // unrolled, the loads of four tiles of more than 64 features crowd the registers (d = 128, fp32, 4000 keys: a layer 208 -> 302 us)
#pragma unroll (HD <= 64 ? 4 : 1)
            for (int tt = 0; tt < 4; ++tt) add_values(tt, 0xffffu, std::true_type{});
        } else {
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                if (t0 + tt >= n_tiles) break;
                add_values(tt, (uint32_t)(seen >> (tt * 16)) & 0xffffu, std::false_type{});
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    for (int d = 32; d > 0; d >>= 1) l += __shfl_xor(l, d);
    if (lane == 0) { wm[wave] = m; wl[wave] = l; }
#pragma unroll
    for (int f = 0; f < FD; ++f)
        if (lane + f * 64 < HD) wo[wave][lane + f * 64] = o[f];
    __syncthreads();
    float M = -INFINITY;
    for (int w = 0; w < 4; ++w) M = fmaxf(M, wm[w]);
    float L = 0.f, f4[4];
    for (int w = 0; w < 4; ++w) { f4[w] = wm[w] == -INFINITY ? 0.f : __expf(wm[w] - M); L += wl[w] * f4[w]; }
    for (int i = threadIdx.x; i < HD; i += 256) {
        float acc = 0.f;
        for (int w = 0; w < 4; ++w) acc += wo[w][i] * f4[w];
        out[((size_t)r * Hq + hq) * HD + i] = from_f<T>(acc / L);
    }
}

template <typename T>
static void attn_generic_t(hipStream_t s, const void *q, void *out, const void *pool_layer, const KvGeom &kg,
                           const RowMeta &rm, const SeqState &st, int Hq, int max_rows)
{
    dim3 grid(Hq, max_rows), block(256);
    switch (kg.head_dim) {
    case 32: hipLaunchKernelGGL((attn_generic_k<T, 32>), grid, block, 0, s, (const T *)q, (T *)out, (const T *)pool_layer, kg, rm, st, Hq); break;
    case 64: hipLaunchKernelGGL((attn_generic_k<T, 64>), grid, block, 0, s, (const T *)q, (T *)out, (const T *)pool_layer, kg, rm, st, Hq); break;
    case 96: hipLaunchKernelGGL((attn_generic_k<T, 96>), grid, block, 0, s, (const T *)q, (T *)out, (const T *)pool_layer, kg, rm, st, Hq); break;
    default: hipLaunchKernelGGL((attn_generic_k<T, 128>), grid, block, 0, s, (const T *)q, (T *)out, (const T *)pool_layer, kg, rm, st, Hq); break;
    }
}

void launch_attn_generic(hipStream_t s, int dtype, const void *q, void *out, const void *pool_layer, const KvGeom &kg,
                         const RowMeta &rm, const SeqState &st, int n_q_heads, int max_rows)
{
    if (dtype == 0) attn_generic_t<float>(s, q, out, pool_layer, kg, rm, st, n_q_heads, max_rows);
    else attn_generic_t<bf16_t>(s, q, out, pool_layer, kg, rm, st, n_q_heads, max_rows);
}

// ------------------------------------------------------------------------------------------------ vocabulary reduction
// Per block row: arg-max (lowest index on ties), and the confidence of Sec. 3.4: (1) softmax probability of the
// arg-max token = 1 / sum exp(z - max); (2) 1 - H / log|V| with H = log S - (sum e^{z-m} (z-m)) / S.
__global__ __launch_bounds__(256) void lm_reduce_k(const float *logits, int V, int32_t *ids, float *conf, int conf_fn,
                                                   const int32_t *p_rows)
{
    int row = blockIdx.x;
    if (row >= *p_rows) return;
    const float *z = logits + (size_t)row * V;
    __shared__ float sm[4];
    __shared__ int si[4];
    __shared__ float red[4];
    float m = -INFINITY;
    int arg = 0;   // stays a valid id even if every logit is NaN
    for (int v = threadIdx.x; v < V; v += 256) {
        float t = z[v];
        if (t > m) { m = t; arg = v; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        float om = __shfl_xor(m, o);
        int oa = __shfl_xor(arg, o);
        if (om > m || (om == m && oa < arg)) { m = om; arg = oa; }
    }
    if ((threadIdx.x & 63) == 0) { sm[threadIdx.x >> 6] = m; si[threadIdx.x >> 6] = arg; }
    __syncthreads();
    m = sm[0]; arg = si[0];
    for (int w = 1; w < 4; ++w)
        if (sm[w] > m || (sm[w] == m && si[w] < arg)) { m = sm[w]; arg = si[w]; }
    float S = 0.f, E = 0.f;
    for (int v = threadIdx.x; v < V; v += 256) {
        float dlt = z[v] - m, e = __expf(dlt);
        S += e;
        E += e * dlt;
    }
    S = block_sum(S, red);
    E = block_sum(E, red);
    if (threadIdx.x == 0) {
        ids[row] = arg;
        conf[row] = conf_fn == 0 ? 1.0f / S : 1.0f - (logf(S) - E / S) / logf((float)V);
    }
}

void launch_lm_reduce(hipStream_t s, const float *logits, int V, int32_t *ids, float *conf, int conf_fn,
                      const int32_t *p_rows, int max_rows)
{
    hipLaunchKernelGGL(lm_reduce_k, dim3(max_rows), dim3(256), 0, s, logits, V, ids, conf, conf_fn, p_rows);
}

// ------------------------------------------------------------------------------------------------ acceptance
// gamma_tau (Sec. 3.4): the largest j in 1..D whose cumulative product of confidences is >= tau, at least 1.
// The product is a float product taken left to right.  rule 1: leading positions whose own confidence is >= tau.
// Position j of sequence b: the count is the same in every position's thread, and stored by the first.
__device__ inline void accept_row(const SeqState &st, const int32_t *ids, const float *conf, int b, int D, int j, float tau, int rule, int32_t *ids_out, int32_t *count_out,
                                  float *conf_out)
{
    int best = 1;
    if (rule == 0) {
        float prod = 1.0f;
        for (int i = 1; i <= D; ++i) {
            prod = prod * conf[i - 1];
            if (prod >= tau && i > best) best = i;
        }
    } else {
        int i = 0;
        while (i < D && conf[i] >= tau) ++i;
        if (i > best) best = i;
    }
    if (j == 0) { st.last_count[b] = best; count_out[b] = best; }
    st.last_ids[b * D + j] = ids[j];
    ids_out[b * D + j] = ids[j];
    if (conf_out) conf_out[b * D + j] = conf[j];
}

__global__ void accept_k(SeqState st, const int32_t *ids_rows, const float *conf_rows, int B, int D, float tau, int rule,
                         int32_t *ids_out, int32_t *count_out, float *conf_out)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x, b = e / D;
    if (b < B) accept_row(st, ids_rows + b * D, conf_rows + b * D, b, D, e % D, tau, rule, ids_out, count_out, conf_out);
}

// Vocabulary reduction and acceptance of one sequence's D rows in one launch, for small vocabularies: 1024 threads in equal parts of the rows (a
// wavefront at least), each part as lm_reduce_k.  V = 4096, D = 4: 8.7 + 3.1 us as two launches, 5.8 here.  The line is by the threads of a row: with D up to 8 (two
// wavefronts a row or more) one launch is faster at every V measured, us a step saved with one / 64 sequences: D = 1, V = 16384 20 / 21, D = 4 13 / 16, D = 8, V = 4096 3.2 / 3.5, 16384 6 / 20;
// with one wavefront a row it reads the row for longer than the launch costs: D = 9 and 16, V = 1000 2.5 / 2.7, 2048 0.9 / 2, 4096 -0.7 / -0.5, 8192 -4 / -1, 16384 -14 / 2.
__global__ __launch_bounds__(1024) void lm_accept_k(const float *logits, int V, int conf_fn, SeqState st, int D, int parts, float tau, int rule, int32_t *ids_out,
                                                    int32_t *count_out, float *conf_out)
{
    __shared__ float sm[16], ss[16], se[16], conf[MAX_D];
    __shared__ int sa[16], ids[MAX_D];
    const int tpr = 1024 / parts, row = threadIdx.x / tpr, t = threadIdx.x % tpr, wave = threadIdx.x >> 6, wpr = tpr >> 6, w0 = row * wpr, b = blockIdx.x;
    const bool live = row < D;
    const float *z = logits + (size_t)(b * D + (live ? row : 0)) * V;
    constexpr int U = 16;
    float m = -INFINITY, x[U];
    int arg = 0;   // stays a valid id even if every logit is NaN
    for (int v0 = t; v0 < V; v0 += U * tpr) {
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = v0 + u * tpr < V ? z[v0 + u * tpr] : -INFINITY;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (x[u] > m) { m = x[u]; arg = v0 + u * tpr; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        float om = __shfl_xor(m, o);
        int oa = __shfl_xor(arg, o);
        if (om > m || (om == m && oa < arg)) { m = om; arg = oa; }
    }
    if ((threadIdx.x & 63) == 0) { sm[wave] = m; sa[wave] = arg; }
    __syncthreads();
    m = sm[w0]; arg = sa[w0];
    for (int w = 1; w < wpr; ++w)
        if (sm[w0 + w] > m || (sm[w0 + w] == m && sa[w0 + w] < arg)) { m = sm[w0 + w]; arg = sa[w0 + w]; }
    float S = 0.f, E = 0.f;
    for (int v0 = t; v0 < V; v0 += U * tpr) {
        if (V > U * tpr) {   // else the values are still there
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = v0 + u * tpr < V ? z[v0 + u * tpr] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (v0 + u * tpr < V) {
                float dlt = x[u] - m, e = __expf(dlt);
                S += e;
                E += e * dlt;
            }
    }
    for (int o = 32; o > 0; o >>= 1) { S += __shfl_xor(S, o); E += __shfl_xor(E, o); }
    if ((threadIdx.x & 63) == 0) { ss[wave] = S; se[wave] = E; }
    __syncthreads();
    if (live && t == 0) {
        S = 0.f; E = 0.f;
        for (int w = 0; w < wpr; ++w) { S += ss[w0 + w]; E += se[w0 + w]; }
        ids[row] = arg;
        conf[row] = conf_fn == 0 ? 1.0f / S : 1.0f - (logf(S) - E / S) / logf((float)V);
    }
    __syncthreads();
    if (threadIdx.x < D) accept_row(st, ids, conf, b, D, threadIdx.x, tau, rule, ids_out, count_out, conf_out);
}

bool lm_accept_applies(int V, int D) { return V <= (D <= 8 ? 16384 : 2048); }

void launch_lm_accept(hipStream_t s, const float *logits, int V, int conf_fn, const SeqState &st, int B, int D, float tau, int rule, int32_t *ids_out,
                      int32_t *count_out, float *conf_out)
{
    int parts = 1;
    while (parts < D) parts *= 2;
    hipLaunchKernelGGL(lm_accept_k, dim3(B), dim3(1024), 0, s, logits, V, conf_fn, st, D, parts, tau, rule, ids_out, count_out, conf_out);
}

void launch_accept(hipStream_t s, const SeqState &st, const int32_t *ids_rows, const float *conf_rows, int B, int D,
                   float tau, int rule, int32_t *ids_out, int32_t *count_out, float *conf_out)
{
    hipLaunchKernelGGL(accept_k, dim3((B * D + 63) / 64), dim3(64), 0, s, st, ids_rows, conf_rows, B, D, tau, rule, ids_out, count_out, conf_out);
}

// ------------------------------------------------------------------------------------------------ commit
// c <- n (the pending K/V, already in place, become cache); the accepted tokens become the pending tokens;
// n <- n + count; the page table grows so that every position < n is backed.
__global__ void commit_k(SeqState st, int B, int D, const int32_t *ids_ovr, const int32_t *cnt_ovr, int paged, int n_pages,
                         int pages_per_seq, int V)
{
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int32_t *ids = ids_ovr ? ids_ovr + b * D : st.last_ids + b * D;
    int cnt = cnt_ovr ? cnt_ovr[b] : st.last_count[b];
    if (cnt < 1 || cnt > D) { atomicOr(&st.alloc[1], 2); cnt = cnt < 1 ? 1 : D; }
    int n = st.n[b], n_new = n + cnt;
    int need = (n_new + PAGE - 1) / PAGE - st.pages_backed[b];
    if (need > 0) {
        if (!paged || st.pages_backed[b] + need > pages_per_seq) { atomicOr(&st.alloc[1], 1); return; }
        int first = atomicAdd(&st.alloc[0], need);
        if (first + need > n_pages) { atomicOr(&st.alloc[1], 1); return; }
        for (int i = 0; i < need; ++i) st.page_table[(size_t)b * pages_per_seq + st.pages_backed[b] + i] = first + i;
        st.pages_backed[b] += need;
    }
    for (int i = 0; i < cnt; ++i) {
        int id = ids[i];
        if (id < 0 || id >= V) { atomicOr(&st.alloc[1], 4); id = 0; }   // an override token outside the vocabulary
        st.pend_tok[b * D + i] = id;
    }
    st.last_tok[b] = st.pend_tok[b * D + cnt - 1];
    st.c[b] = n;
    st.n[b] = n_new;
}

void launch_commit(hipStream_t s, const SeqState &st, int B, int D, const int32_t *ids_ovr, const int32_t *cnt_ovr,
                   int paged, int n_pages, int pages_per_seq, int V)
{
    hipLaunchKernelGGL(commit_k, dim3((B + 63) / 64), dim3(64), 0, s, st, B, D, ids_ovr, cnt_ovr, paged, n_pages, pages_per_seq, V);
}

// ------------------------------------------------------------------------------------------------ debug read-back
template <typename T>
__global__ void read_kv_k(const T *pool, KvGeom kg, SeqState st, int seq, int kvh, int pos0, int count, float *k_out, float *v_out)
{
    int d = kg.head_dim;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < count * d; e += gridDim.x * blockDim.x) {
        int pos = pos0 + e / d, i = e % d;
        int page, slot;
        if (pos0 < 0) { page = kg.staging_base + seq; slot = e / d; }   // the block rows' staging tile
        else { page = st.page_table[(size_t)seq * kg.pages_per_seq + pos / PAGE]; slot = pos % PAGE; }
        const T *Kb = pool + kg.tile(page, kvh), *Vb = Kb + PAGE * d;
        k_out[e] = to_f<T>(Kb[k_off(slot, i)]);
        v_out[e] = to_f<T>(Vb[v_off(slot, i)]);
    }
}

void launch_read_kv(hipStream_t s, int dtype, const void *pool_layer, const KvGeom &kg, const SeqState &st, int seq,
                    int kvh, int pos0, int count, float *k_out, float *v_out)
{
    int blocks = (count * kg.head_dim + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    if (dtype == 0) hipLaunchKernelGGL(read_kv_k<float>, dim3(blocks), dim3(256), 0, s, (const float *)pool_layer, kg, st, seq, kvh, pos0, count, k_out, v_out);
    else hipLaunchKernelGGL(read_kv_k<bf16_t>, dim3(blocks), dim3(256), 0, s, (const bf16_t *)pool_layer, kg, st, seq, kvh, pos0, count, k_out, v_out);
}

}  // namespace sdlm
