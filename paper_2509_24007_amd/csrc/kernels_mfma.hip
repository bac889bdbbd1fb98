// Matrix-core (MFMA) GEMMs of the bf16 mode: the QKV / O / gate-up / down projections and the LM head with its
// fused vocabulary reduction.  These are the path's only true dense contractions.
//
// Y[r, n] = sum_k X[r, k] W[n, k], R activation rows (8 .. 2048) against N weight rows: every weight byte is
// needed exactly once per step, so the kernels are organised around streaming W from HBM.
//   * W is repacked once (sdlm_init_weights) into the operand order of v_mfma_f32_32x32x16_bf16: tile (n/32,
//     k/16) is 64 lanes x 8 bf16 = 1 KB contiguous and the tiles of one 32-row band follow each other along k,
//     so a wavefront's operand stream is a plain contiguous run, loaded global -> registers with 16-byte loads
//     and never staged in LDS (no other wavefront of the workgroup needs the same weights).
//   * The weight tile is the A operand (M = 32 output features), the activation rows are the B operand
//     (N = 32 rows).  A workgroup is 4 wavefronts; each owns NT bands of output features and all of them
//     share the MT*32 activation rows of the workgroup, which are staged in LDS (64-deep k slices, double
//     buffered, rows padded to 144 bytes so that the 16-byte operand reads do not collide on banks).
//   * Skinny problems (few rows, few output features) are split along k; the partial sums go to a scratch
//     slab per split and are added in a fixed order by the consumer, so results do not depend on timing.
//   * Workgroup ids are remapped so that the row blocks of one weight band run on the same XCD and share its L2,
//     and so that the row blocks which may be empty come last in the grid (see the kernel).
#include "mfma.hpp"

namespace sdlm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int XS_STRIDE = 72;   // bf16 elements per LDS row of the activation slice (64 + 8 padding)
constexpr int ZT_STRIDE = 68;   // floats per LDS row of a wavefront's 32 x 64 logits (64 + 4 padding)

bool mfma_supported(const sdlm_model_cfg *m)
{
    return m->dtype == 1 && m->head_dim == 128 && m->hidden % 64 == 0 && m->ffn % 64 == 0 &&
           (m->n_q_heads * m->head_dim) % 64 == 0 && m->n_q_heads / m->n_kv_heads <= 64;
}
size_t mfma_pad_n(size_t N) { return (N + 31) / 32 * 32; }
size_t mfma_packed_elems(bool packed, size_t N, size_t K) { return (packed ? mfma_pad_n(N) : N) * K; }

// ------------------------------------------------------------------------------------------------ weight packing
// dst tile order: [n/32][k/16][lane][8] with lane = (n % 32) + 32 * ((k % 16) / 8).
__global__ void pack_mfma_k(bf16_t *dst, const bf16_t *src, int N, int K, int dst_row0, int interleave)
{
    const int KS = K / 16;
    size_t g = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 8-element group
    size_t total = (size_t)((N + 31) / 32) * KS * 64;
    if (g >= total) return;
    int lane = (int)(g & 63);
    size_t t = g >> 6;
    int ks = (int)(t % KS), nt = (int)(t / KS);
    int n = nt * 32 + (lane & 31), k = ks * 16 + (lane >> 5) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (n < N) v = *(const uint4 *)(src + (size_t)n * K + k);
    int dtile = interleave == 0 ? dst_row0 / 32 + nt : 2 * nt + (interleave - 1);
    *(uint4 *)(dst + (((size_t)dtile * KS + ks) * 64 + lane) * 8) = v;
}

void launch_pack_mfma(hipStream_t s, void *dst, const void *src, int N, int K, int dst_row0, int, int interleave)
{
    size_t total = (size_t)((N + 31) / 32) * (K / 16) * 64;
    hipLaunchKernelGGL(pack_mfma_k, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (bf16_t *)dst, (const bf16_t *)src, N, K, dst_row0, interleave);
}

// ------------------------------------------------------------------------------------------------ GEMM
struct MfmaArgs {
    const bf16_t *X, *Wp, *bias;
    float *Yf;          // STORE_F32 / RESID destination, or split-k slabs
    bf16_t *Yt;         // SWIGLU destination
    float *logits;      // LM head: optional [rows, N] logits
    float4 *lm_part;    // LM head: [n_blocks][max_rows] partial (max, sum, entropy sum, argmax bits)
    const int32_t *pR;
    int max_rows, N, K, n_tiles, n_blocks, m_blocks, splits, stages_per_split, n_out;   // n_out: row length of the destination
    int m_sure;         // row blocks below this index certainly hold rows; they come first in the grid
    int rows_sure;      // rows below this index certainly exist (host-known lower bound of the device row count)
    size_t slab;        // elements between split-k slabs
    float scale, eps;
    const bf16_t *gain; // steps of at most 16 rows: see "norms inside the products"
    bf16_t *xg;
    float *ssq;
};

enum { EPI_LMHEAD = 4 };

__device__ inline float silu_f(float v) { return v / (1.0f + __expf(-v)); }

// The largest tile keeps two register sets of weights instead of three so that accumulators + operands fit in 256
// registers: two workgroups then share a compute unit and one's barrier and load waits are covered by the other.
template <int MT, int NT> constexpr int w_sets() { return (MT >= 4) ? 2 : 3; }

// WV wavefronts per workgroup: 4, or 8 (a 128-row x 512-column tile whose activation slice is staged once for eight
// wavefronts instead of once for four: fewer bytes through the compute unit's load path per MFMA).
// KH = 2: the wavefronts form two halves that take a half of k each (gate/up with few column blocks, see refine_gateup); the halves'
// sums meet in LDS before the epilogue.  The columns of a workgroup are then those of WV / 2 wavefronts.
template <int MT, int NT, int EPI, int WV = 4, int KH = 1>
__global__ __launch_bounds__(WV * 64, (WV == 8 || KH == 2 ? 1 : (MT == 4 ? 2 : 1))) void gemm_mfma_k(MfmaArgs a)
{
    static_assert(WV == 4 || (WV == 8 && MT % 2 == 0), "eight wavefronts stage two 32-row sub-tiles per load round");
    // the activation slices; the LM head's epilogue afterwards turns its logits around in the same memory
    constexpr size_t XS_BYTES = sizeof(bf16_t) * 2 * KH * MT * 32 * XS_STRIDE, ZT_BYTES = EPI == EPI_LMHEAD ? sizeof(float) * WV * 32 * ZT_STRIDE : 0;
    __shared__ __attribute__((aligned(16))) unsigned char smem[XS_BYTES > ZT_BYTES ? XS_BYTES : ZT_BYTES];
    auto Xs = reinterpret_cast<bf16_t (*)[KH * MT * 32][XS_STRIDE]>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps the weight stream's base in SGPRs
    // workgroup id -> tile.  The grid has two parts: the row blocks that certainly hold rows (mblk < m_sure), then the
    // others, which usually exit at once; mixing them would leave the compute units that draw an empty block idle.
    // Within a part, ids that land on one XCD (id % 8) get consecutive tiles, the row blocks of one weight band first.
    const int n_first = a.n_blocks * a.splits * a.m_sure, first8 = (n_first + 7) & ~7;
    int mblk, rest;
    if ((int)blockIdx.x < first8) {
        const int per = first8 >> 3, t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
        if (t >= n_first) return;
        mblk = t % a.m_sure; rest = t / a.m_sure;
    } else {
        const int bid = blockIdx.x - first8, m_rest = a.m_blocks - a.m_sure;
        const int per = (gridDim.x - first8) >> 3, t = (bid & 7) * per + (bid >> 3);
        if (t >= a.n_blocks * a.splits * m_rest) return;
        mblk = a.m_sure + t % m_rest; rest = t / m_rest;
    }
    const int split = rest % a.splits, nblk = rest / a.splits;
    const int m0 = mblk * MT * 32;
    // A row block that lies entirely below the host-known row bound does not wait for the device-side row count: its
    // first operand requests go out at once (the count is one more memory round trip at the head of the kernel).
    const int R = m0 + MT * 32 <= a.rows_sure ? a.rows_sure : min(*a.pR, a.max_rows);
    if (m0 >= R) return;
    const int KS = a.K >> 4, S = a.K >> 6;
    constexpr int CW = WV / KH;                                    // wavefronts side by side
    const int cwave = wave % CW, half = KH == 1 ? 0 : wave / CW;   // column and k half of this wavefront
    const int s_first = split * a.stages_per_split, s_count = min(S - s_first, a.stages_per_split);   // this split's slices; KH = 2: an even number
    const int s_begin = s_first + half * (s_count / KH), s_end = s_begin + s_count / KH;
    if (s_begin >= s_end) return;

    // Addresses are (wave-uniform base) + (32-bit per-lane offset): the loads then take their base from SGPRs and
    // no address register is ever the destination of a load still in flight.
    const bf16_t *wp[NT];
    int ntile[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        ntile[nt] = (nblk * CW + cwave) * NT + nt;
        int tl = min(ntile[nt], a.n_tiles - 1);
        wp[nt] = a.Wp + ((size_t)tl * KS) * 512;
    }
    const uint32_t wlane = lane * 8;
    // activation slice: MT*32 rows x 64 k = MT*256 16-byte chunks, XC per thread (a round of loads covers XR rows); with two k
    // halves a slice of each, rounds alternating between them
    constexpr int XR = WV * 8, XC = KH * MT * 32 / XR;
    const int xrow = tid >> 3, xchunk = tid & 7;
    uint32_t xoff[XC];
#pragma unroll
    for (int i = 0; i < XC; ++i) xoff[i] = (uint32_t)min(m0 + i / KH * XR + xrow, R - 1) * (uint32_t)a.K + xchunk * 8 + (i % KH) * (s_count / KH) * 64;
    constexpr auto xs_row = [](int i) { return i % KH * (MT * 32) + i / KH * XR; };   // LDS row where load round i begins

    f32x16 acc[NT][MT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[nt][mt][v] = 0.f;

    // Software pipeline.  Small tiles (MT < 4): three rotating weight register sets, the weights of slice s+2 and the
    // activations of slice s+1 are requested at the top of slice s (the loop is unrolled by three so that the sets keep
    // static names).  128-row tiles: two weight sets and one activation operand set, so that accumulators + operands
    // fit in 256 registers and two workgroups share a compute unit; the loads of slice s+1 are spread over slice s.
    // In both, the activations go registers -> LDS at the bottom of the slice, and activation loads are issued before
    // weight loads: the counter that orders returns is in program order, so waiting for the (L2-hot) activations
    // leaves the (HBM) weight loads in flight.
    bf16x8 w0[NT][4], w1[NT][4], w2[w_sets<MT, NT>() == 3 ? NT : 1][4];
    u32x4 xr[XC];
    const int s_last = s_end - 1;
#define SDLM_LOAD_W(dst, stage)                                                                                   \
    {                                                                                                             \
        const size_t so_ = (size_t)min((stage), s_last) * 4 * 512;                                                \
        /* in the order the next slice's k-steps consume them */                                                  \
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks)                                                         \
            _Pragma("unroll") for (int nt = 0; nt < NT; ++nt) dst[nt][ks] = *(const bf16x8 *)(wp[nt] + so_ + ks * 512 + wlane); \
    }
#define SDLM_LOAD_X(stage)                                                                                        \
    {                                                                                                             \
        const size_t xo_ = (size_t)(min((stage), s_last) - half * (s_count / KH)) * 64;                                                     \
        _Pragma("unroll") for (int i = 0; i < XCA_; ++i) xr[i] = *(const u32x4 *)(a.X + xo_ + xoff[i]);          \
    }
    constexpr int WSETS = w_sets<MT, NT>();
    const int brow = lane & 31, bk = (lane >> 5) * 8, lrow = half * (MT * 32) + brow;   // lrow: LDS row of the lane's operand
/* ---- three weight sets (small tiles): one k-step = request the LDS operands of the next k-step, run this k-step's
   MFMAs, and pin that order; the slice's global loads are issued at its top */
#define SDLM_KSTEP(WC, ks, has_next)                                                                              \
    {                                                                                                             \
        if (has_next) {                                                                                           \
            _Pragma("unroll") for (int mt = 0; mt < MTA_; ++mt)                                                  \
                bn_[mt] = *(const bf16x8 *)&Xs[buf][mt * 32 + lrow][((ks) + 1) * 16 + bk];                        \
        }                                                                                                         \
        _Pragma("unroll") for (int mt = 0; mt < MTA_; ++mt)                                                      \
            _Pragma("unroll") for (int nt = 0; nt < NT; ++nt)                                                    \
                acc[nt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(WC[nt][ks], bc_[mt], acc[nt][mt], 0, 0, 0); \
        __builtin_amdgcn_sched_group_barrier(0x100, (has_next) ? MTA_ : 0, 0);                                    \
        __builtin_amdgcn_sched_group_barrier(0x008, MTA_ * NT, 0);                                                \
        _Pragma("unroll") for (int mt = 0; mt < MTA_; ++mt) bc_[mt] = bn_[mt];                                   \
    }
#define SDLM_STAGE3(WC, WN, stage)                                                                                \
    {                                                                                                             \
        SDLM_LOAD_X((stage) + 1);                                                                                 \
        SDLM_LOAD_W(WN, (stage) + 2);                                                                             \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        bf16x8 bc_[MT], bn_[MT];                                                                                  \
        _Pragma("unroll") for (int mt = 0; mt < MTA_; ++mt) bc_[mt] = *(const bf16x8 *)&Xs[buf][mt * 32 + lrow][bk]; \
        __builtin_amdgcn_sched_group_barrier(0x100, MTA_, 0);                                                     \
        SDLM_KSTEP(WC, 0, 1) SDLM_KSTEP(WC, 1, 1) SDLM_KSTEP(WC, 2, 1) SDLM_KSTEP(WC, 3, 0)                       \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        _Pragma("unroll") for (int i = 0; i < XCA_; ++i) *(u32x4 *)&Xs[buf ^ 1][xs_row(i) + xrow][xchunk * 8] = xr[i]; \
        buf ^= 1;                                                                                                 \
        __syncthreads();                                                                                          \
    }
/* ---- two weight sets (128-row tiles): a single activation operand set bq_; each fragment is re-read in place
   right after the MFMAs that used it (slot = the MFMAs of one 32-row sub-tile at one k-step).  The slice is pipelined
   across its own boundary so that the MFMA stream never waits for LDS:
     k-steps 0, 1   MFMAs; the weight loads of the next slice dealt out over the slots (the load unit never holds the
                    wavefront up)
     publish        the activations of the next slice (requested a whole slice ago) go registers -> the other LDS buffer
     k-step 2       MFMAs; the activation loads of the slice after next, one per slot
     barrier        the other buffer is complete; nobody reads this slice's buffer after k-step 2 (the fragments of
                    k-step 3 are already in registers)
     k-step 3       MFMAs; each fragment register is refilled with the next slice's first fragment from the other buffer
   The next slice therefore starts with its operands in registers, and the LDS writes complete under k-step 2. */
#define SDLM_SLOT(WC, ks, mt, SRC, koff, vm)                                                                      \
    if constexpr ((mt) < MTA_) {                                                                                  \
        _Pragma("unroll") for (int nt = 0; nt < NT; ++nt)                                                        \
            acc[nt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(WC[nt][ks], bq_[mt], acc[nt][mt], 0, 0, 0);     \
        bq_[mt] = *(const bf16x8 *)&Xs[SRC][(mt) * 32 + lrow][(koff) + bk];                                       \
        __builtin_amdgcn_sched_group_barrier(0x020, (vm), 0);                                                     \
        __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);                                                       \
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                                        \
    }
/* weight loads of slot i of the 2 MTA_ slots of k-steps 0 and 1: 4 NT loads spread evenly */
#define SDLM_WVM(i) (((i) + 1) * 4 * NT / (2 * MTA_) - (i) * 4 * NT / (2 * MTA_))
#define SDLM_KSTEP2(WC, ks, SRC, koff, VM)                                                                        \
    SDLM_SLOT(WC, ks, 0, SRC, koff, VM(0)) SDLM_SLOT(WC, ks, 1, SRC, koff, VM(1)) SDLM_SLOT(WC, ks, 2, SRC, koff, VM(2)) \
    SDLM_SLOT(WC, ks, 3, SRC, koff, VM(3)) SDLM_SLOT(WC, ks, 4, SRC, koff, VM(4)) SDLM_SLOT(WC, ks, 5, SRC, koff, VM(5)) \
    SDLM_SLOT(WC, ks, 6, SRC, koff, VM(6)) SDLM_SLOT(WC, ks, 7, SRC, koff, VM(7))
#define SDLM_VM_W0(mt) SDLM_WVM(mt)
#define SDLM_VM_W1(mt) SDLM_WVM(MTA_ + (mt))
#define SDLM_VM_ONE(mt) ((mt) < XCA_ / KH ? KH : 0)
#define SDLM_VM_NONE(mt) 0
#define SDLM_STAGE2(WC, WN, stage)                                                                                \
    {                                                                                                             \
        SDLM_LOAD_W(WN, (stage) + 1);                                                                             \
        SDLM_KSTEP2(WC, 0, buf, 16, SDLM_VM_W0) SDLM_KSTEP2(WC, 1, buf, 32, SDLM_VM_W1)                           \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        _Pragma("unroll") for (int i = 0; i < XCA_; ++i) *(u32x4 *)&Xs[buf ^ 1][xs_row(i) + xrow][xchunk * 8] = xr[i]; \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        SDLM_LOAD_X((stage) + 2);                                                                                 \
        SDLM_KSTEP2(WC, 2, buf, 48, SDLM_VM_ONE)                                                                  \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        __syncthreads();                                                                                          \
        SDLM_KSTEP2(WC, 3, buf ^ 1, 0, SDLM_VM_NONE)                                                              \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        buf ^= 1;                                                                                                 \
    }
/* The whole k loop for a row block of which only the first MTA_VALUE 32-row sub-tiles hold rows (the last block of
   a launch is usually ragged): the empty sub-tiles' loads, LDS traffic and MFMAs are not issued at all.  Full
   triples (pairs) of slices run without any branch inside the loop (a conditional stage would make the compiler
   drain all outstanding loads at the loop head); the remaining slices are peeled. */
#define SDLM_MAIN(MTA_VALUE)                                                                                      \
    {                                                                                                             \
        constexpr int MTA_ = MTA_VALUE, XCA_ = KH * ((MTA_VALUE * 32 + XR - 1) / XR);   /* live sub-tiles; load rounds that cover them */ \
        int buf = 0;                                                                                              \
        SDLM_LOAD_X(s_begin);                                                                                     \
        SDLM_LOAD_W(w0, s_begin);                                                                                 \
        if (WSETS == 3) SDLM_LOAD_W(w1, s_begin + 1);                                                             \
        _Pragma("unroll") for (int i = 0; i < XCA_; ++i) *(u32x4 *)&Xs[0][xs_row(i) + xrow][xchunk * 8] = xr[i];    \
        __syncthreads();                                                                                          \
        bf16x8 bq_[MT];                                                                                           \
        if constexpr (WSETS == 2) {   /* the pipelined slice expects its first fragments and the next activations */ \
            SDLM_LOAD_X(s_begin + 1);                                                                             \
            _Pragma("unroll") for (int mt = 0; mt < MTA_; ++mt) bq_[mt] = *(const bf16x8 *)&Xs[0][mt * 32 + lrow][bk]; \
        }                                                                                                         \
        int s = s_begin;                                                                                          \
        if constexpr (WSETS == 3) {                                                                               \
            for (; s + 3 <= s_end; s += 3) {                                                                      \
                SDLM_STAGE3(w0, w2, s)                                                                            \
                SDLM_STAGE3(w1, w0, s + 1)                                                                        \
                SDLM_STAGE3(w2, w1, s + 2)                                                                        \
            }                                                                                                     \
            if (s < s_end) {                                                                                      \
                SDLM_STAGE3(w0, w2, s)                                                                            \
                if (s + 1 < s_end) SDLM_STAGE3(w1, w0, s + 1)                                                     \
            }                                                                                                     \
        } else {                                                                                                  \
            for (; s + 2 <= s_end; s += 2) {                                                                      \
                SDLM_STAGE2(w0, w1, s)                                                                            \
                SDLM_STAGE2(w1, w0, s + 1)                                                                        \
            }                                                                                                     \
            if constexpr (MT < 8) {   /* 256-row tiles: an even number of slices */                                \
                if (s < s_end) SDLM_STAGE2(w0, w1, s)                                                             \
            }                                                                                                     \
        }                                                                                                         \
    }
    const int mt_act = min(MT, (R - m0 + 31) >> 5);   // >= 1: m0 < R
    if constexpr (MT == 8) {
        if (mt_act == 8) SDLM_MAIN(8) else if (mt_act == 7) SDLM_MAIN(7) else if (mt_act == 6) SDLM_MAIN(6) else if (mt_act == 5) SDLM_MAIN(5)
        else if (mt_act == 4) SDLM_MAIN(4) else if (mt_act == 3) SDLM_MAIN(3) else if (mt_act == 2) SDLM_MAIN(2) else SDLM_MAIN(1)
    } else if constexpr (MT == 6) {
        if (mt_act == 6) SDLM_MAIN(6) else if (mt_act == 5) SDLM_MAIN(5) else if (mt_act == 4) SDLM_MAIN(4) else if (mt_act == 3) SDLM_MAIN(3)
        else if (mt_act == 2) SDLM_MAIN(2) else SDLM_MAIN(1)
    } else if constexpr (MT == 4) {
        if (mt_act == 4) SDLM_MAIN(4) else if (mt_act == 3) SDLM_MAIN(3) else if (mt_act == 2) SDLM_MAIN(2) else SDLM_MAIN(1)
    } else if constexpr (MT == 2) {
        if (mt_act == 2) SDLM_MAIN(2) else SDLM_MAIN(1)
    } else {
        SDLM_MAIN(1)
    }
#undef SDLM_MAIN
#undef SDLM_STAGE3
#undef SDLM_STAGE2
#undef SDLM_KSTEP
#undef SDLM_KSTEP2
#undef SDLM_SLOT
#undef SDLM_WVM
#undef SDLM_VM_W0
#undef SDLM_VM_W1
#undef SDLM_VM_ONE
#undef SDLM_VM_NONE
#undef SDLM_LOAD_W
#undef SDLM_LOAD_X

    if constexpr (KH == 2) {
        // each half finishes every other 32-row sub-tile: it hands the other ones over and adds what it is handed
        static_assert(KH == 1 || (MT + 1) / 2 * NT * 4096 * WV <= (int)XS_BYTES, "the halves' exchange reuses the activation slices' memory");
        float *px = reinterpret_cast<float *>(smem);
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            if ((mt & 1) != half && mt < mt_act)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *(float4 *)&px[((((wave * ((MT + 1) / 2) + mt / 2) * NT + nt) * 4 + q) * 64 + lane) * 4] =
                            make_float4(acc[nt][mt][q * 4], acc[nt][mt][q * 4 + 1], acc[nt][mt][q * 4 + 2], acc[nt][mt][q * 4 + 3]);
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            if ((mt & 1) == half && mt < mt_act)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 o = *(const float4 *)&px[(((((wave ^ CW) * ((MT + 1) / 2) + mt / 2) * NT + nt) * 4 + q) * 64 + lane) * 4];
                        acc[nt][mt][q * 4] += o.x; acc[nt][mt][q * 4 + 1] += o.y; acc[nt][mt][q * 4 + 2] += o.z; acc[nt][mt][q * 4 + 3] += o.w;
                    }
    }
    // accumulator element v of lane l: output feature 8*(v/4) + 4*(l/32) + v%4 of the tile, activation row l%32
    const int fbase = (lane >> 5) * 4;
    if (EPI == EPI_STORE_F32 || EPI == EPI_RESID) {
        float *dst = a.Yf + (a.splits > 1 ? (size_t)split * a.slab : 0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (ntile[nt] >= a.n_tiles) continue;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                int r = m0 + mt * 32 + brow;
                if (r >= R) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    int n = ntile[nt] * 32 + q * 8 + fbase;
                    if (n >= a.N) continue;
                    float4 v = make_float4(acc[nt][mt][q * 4], acc[nt][mt][q * 4 + 1], acc[nt][mt][q * 4 + 2], acc[nt][mt][q * 4 + 3]);
                    float4 *p = (float4 *)(dst + (size_t)r * a.n_out + n);
                    if (EPI == EPI_STORE_F32) {
                        if (a.bias && split == 0) {
                            v.x += bf16_to_f(a.bias[n]); v.y += bf16_to_f(a.bias[n + 1]);
                            v.z += bf16_to_f(a.bias[n + 2]); v.w += bf16_to_f(a.bias[n + 3]);
                        }
                        *p = v;
                    } else if (a.splits > 1) {
                        *p = v;
                    } else {
                        float4 o = *p;
                        o.x += v.x; o.y += v.y; o.z += v.z; o.w += v.w;
                        *p = o;
                    }
                }
            }
        }
    } else if (EPI == EPI_SWIGLU) {
        // the fused matrix alternates 32-row tiles of gate and up: tiles (2j, 2j+1) belong to features 32j..32j+31
        static_assert(EPI != EPI_SWIGLU || NT == 2, "gate and up tiles must sit in one wavefront");
        const int j = ntile[0] >> 1;
        if (ntile[0] + 1 < a.n_tiles + 1 && ntile[0] < a.n_tiles) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                int r = m0 + mt * 32 + brow;
                if (r >= R || (KH == 2 && (mt & 1) != half)) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    int n = j * 32 + q * 8 + fbase;
                    if (n >= a.N) continue;
                    float o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = silu_f(acc[0][mt][q * 4 + e]) * acc[NT - 1][mt][q * 4 + e];
                    *(uint2 *)(a.Yt + (size_t)r * a.n_out + n) = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
                }
            }
        }
    } else {
        // LM head: logits of this workgroup's 128*NT vocabulary entries -> per-row (max, argmax, sum exp, entropy sum).
        // Logits the caller asked for go through LDS, 32 rows x 64 entries per wavefront at a time, so that a store is 256
        // contiguous bytes of one row: from the accumulators it would be 64 single values 4 V bytes apart, and the address
        // unit takes one cache line at a time.  V = 151936, with logits: h = 2048, 128 rows 200 -> 156 us; h = 3584, 256 rows
        // (V = 152064) 384 -> 314 us; few rows gain nothing (4 rows, h = 1536: 92 -> 91 us).
        __shared__ float sm_m[WV][MT * 32];
        __shared__ int sm_a[WV][MT * 32];
        __shared__ float sm_s[WV][MT * 32], sm_e[WV][MT * 32];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float m = -INFINITY;
            int arg = 0;   // stays a valid id even if every logit is NaN
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    int n = ntile[nt] * 32 + (v >> 2) * 8 + fbase + (v & 3);
                    float z = acc[nt][mt][v] * a.scale;
                    acc[nt][mt][v] = z;
                    if (n < a.N) {
                        if (z > m || (z == m && n < arg)) { m = z; arg = n; }
                    }
                }
            float om = __shfl_xor(m, 32);
            int oa = __shfl_xor(arg, 32);
            if (om > m || (om == m && oa < arg)) { m = om; arg = oa; }
            if (lane < 32) { sm_m[wave][mt * 32 + lane] = m; sm_a[wave][mt * 32 + lane] = arg; }
        }
        __syncthreads();   // also: nobody reads the activation slices any more
        if (a.logits) {
            static_assert(EPI != EPI_LMHEAD || NT == 2, "a row of a wavefront's logits is one store of 64 lanes");
            float *zt = reinterpret_cast<float *>(smem) + wave * 32 * ZT_STRIDE;   // this wavefront's own part: no barrier
            const int n = ntile[0] * 32 + lane;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *(float4 *)&zt[brow * ZT_STRIDE + nt * 32 + q * 8 + fbase] =
                            make_float4(acc[nt][mt][q * 4], acc[nt][mt][q * 4 + 1], acc[nt][mt][q * 4 + 2], acc[nt][mt][q * 4 + 3]);
                const int r0 = m0 + mt * 32, live = min(32, R - r0);
                float *dst = a.logits + (size_t)r0 * a.N + n;
                if (n < a.N)
                    for (int j = 0; j < live; ++j) dst[(size_t)j * a.N] = zt[j * ZT_STRIDE + lane];
            }
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float m = sm_m[0][mt * 32 + brow];
#pragma unroll
            for (int w = 1; w < WV; ++w) m = fmaxf(m, sm_m[w][mt * 32 + brow]);
            float S = 0.f, E = 0.f;
            if (m > -INFINITY) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        int n = ntile[nt] * 32 + (v >> 2) * 8 + fbase + (v & 3);
                        if (n < a.N) {
                            float dlt = acc[nt][mt][v] - m, e = __expf(dlt);
                            S += e;
                            E += e * dlt;
                        }
                    }
            }
            S += __shfl_xor(S, 32);
            E += __shfl_xor(E, 32);
            if (lane < 32) { sm_s[wave][mt * 32 + lane] = S; sm_e[wave][mt * 32 + lane] = E; }
        }
        __syncthreads();
        for (int i = tid; i < MT * 32; i += WV * 64) {
            int r = m0 + i;
            if (r >= R) continue;
            float m = sm_m[0][i];
            int arg = sm_a[0][i];
            float S = sm_s[0][i], E = sm_e[0][i];
            for (int w = 1; w < WV; ++w) {
                if (sm_m[w][i] > m || (sm_m[w][i] == m && sm_a[w][i] < arg)) { m = sm_m[w][i]; arg = sm_a[w][i]; }
                S += sm_s[w][i];
                E += sm_e[w][i];
            }
            a.lm_part[(size_t)nblk * a.max_rows + r] = make_float4(m, S, E, __int_as_float(arg));
        }
    }
}

// x[r, :] += sum over split slabs (fixed order)
__global__ __launch_bounds__(256) void reduce_slabs_k(float *x, const float *part, int splits, size_t slab, int n, const int32_t *pR, int max_rows)
{
    int r = blockIdx.x;
    if (r >= min(*pR, max_rows)) return;
    for (int c = threadIdx.x * 4; c < n; c += 1024) {
        float4 o = *(float4 *)(x + (size_t)r * n + c);
        for (int s = 0; s < splits; ++s) {
            float4 v = *(const float4 *)(part + s * slab + (size_t)r * n + c);
            o.x += v.x; o.y += v.y; o.z += v.z; o.w += v.w;
        }
        *(float4 *)(x + (size_t)r * n + c) = o;
    }
}

// Combine the LM head's per-block partials of one row: overall arg-max (lowest index on ties), and with
// M = max_i m_i:  S = sum_i S_i e^{m_i - M},  E = sum_i e^{m_i - M} (E_i + S_i (m_i - M)).
__global__ __launch_bounds__(256) void lm_combine_k(const float4 *part, int n_blocks, int max_rows, const int32_t *p_rows, int V, int conf_fn,
                                                    int32_t *ids, float *conf)
{
    int r = blockIdx.x;
    if (r >= min(*p_rows, max_rows)) return;
    __shared__ float sm[4];
    __shared__ int sa[4];
    __shared__ float red[4];
    float m = -INFINITY;
    int arg = 0;
    for (int i = threadIdx.x; i < n_blocks; i += 256) {
        float4 p = part[(size_t)i * max_rows + r];
        int a = __float_as_int(p.w);
        if (p.x > m || (p.x == m && a < arg)) { m = p.x; arg = a; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        float om = __shfl_xor(m, o);
        int oa = __shfl_xor(arg, o);
        if (om > m || (om == m && oa < arg)) { m = om; arg = oa; }
    }
    if ((threadIdx.x & 63) == 0) { sm[threadIdx.x >> 6] = m; sa[threadIdx.x >> 6] = arg; }
    __syncthreads();
    m = sm[0]; arg = sa[0];
    for (int w = 1; w < 4; ++w)
        if (sm[w] > m || (sm[w] == m && sa[w] < arg)) { m = sm[w]; arg = sa[w]; }
    float S = 0.f, E = 0.f;
    for (int i = threadIdx.x; i < n_blocks; i += 256) {
        float4 p = part[(size_t)i * max_rows + r];
        float dm = p.x - m, f = __expf(dm);
        S += p.y * f;
        E += f * (p.z + p.y * dm);
    }
    for (int o = 32; o > 0; o >>= 1) { S += __shfl_xor(S, o); E += __shfl_xor(E, o); }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { sm[threadIdx.x >> 6] = S; red[threadIdx.x >> 6] = E; }
    __syncthreads();
    if (threadIdx.x == 0) {
        S = sm[0] + sm[1] + sm[2] + sm[3];
        E = red[0] + red[1] + red[2] + red[3];
        ids[r] = arg;
        conf[r] = conf_fn == 0 ? 1.0f / S : 1.0f - (logf(S) - E / S) / logf((float)V);
    }
}

// ------------------------------------------------------------------------------------------------ gate/up for 17 .. 32 rows
// A step of at most 32 rows cannot split the gate/up projection along k between workgroups (SiLU(gate) * up needs complete
// sums): the tiled kernel above would run it as N/128 workgroups, far too few to keep the weight stream busy.  Here a workgroup
// owns one 32-feature block (its gate tile and its up tile), its four wavefronts each take a quarter of k, and the quarters are
// added in wavefront order through LDS.  Both operands come straight from global memory in the MFMA operand order: the weights as a
// contiguous run, the rows (at most 32 x K, shared by every workgroup, so served by L2) 16 bytes per lane and k step; rows beyond
// the live ones repeat the last row and their results are dropped.  Loads are issued eight k steps at a time into two register
// sets: sixteen k steps (48 KB per wavefront) are in flight before the first MFMA.
constexpr int SK_U = 8, SK_W = 4;   // k steps per register set; wavefronts (measured: eight wavefronts are slower)

__global__ __launch_bounds__(SK_W * 64) void swiglu_skinny32_k(MfmaArgs a)
{
    __shared__ float part[SK_W][2][16][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = blockIdx.x;   // features 32j .. 32j+31: tiles 2j (gate) and 2j+1 (up) of the fused matrix
    const int KS = a.K >> 4, per = (KS + SK_W - 1) / SK_W;
    const int k_begin = wave * per, k_end = min(KS, k_begin + per);
    const bf16_t *wg = a.Wp + ((size_t)(2 * j) * KS) * 512 + lane * 8, *wu = wg + (size_t)KS * 512;
    bf16x8 g0[SK_U], u0[SK_U], x0[SK_U], g1[SK_U], u1[SK_U], x1[SK_U];
#define SDLM_SK_LOAD_W(G, U, kb) \
    _Pragma("unroll") for (int u = 0; u < SK_U; ++u) { \
        const size_t o = (size_t)min((kb) + u, KS - 1) * 512; \
        G[u] = *(const bf16x8 *)(wg + o); U[u] = *(const bf16x8 *)(wu + o); }
#define SDLM_SK_LOAD_X(X, kb) \
    _Pragma("unroll") for (int u = 0; u < SK_U; ++u) X[u] = *(const bf16x8 *)(xp + min((kb) + u, KS - 1) * 16);
#define SDLM_SK_MMA(G, U, X, kb) \
    _Pragma("unroll") for (int u = 0; u < SK_U; ++u) if ((kb) + u < k_end) { \
        ag = __builtin_amdgcn_mfma_f32_32x32x16_bf16(G[u], X[u], ag, 0, 0, 0); \
        au = __builtin_amdgcn_mfma_f32_32x32x16_bf16(U[u], X[u], au, 0, 0, 0); }
    SDLM_SK_LOAD_W(g0, u0, k_begin)   // the weights do not wait for the row count
    if (k_begin + SK_U < k_end) { SDLM_SK_LOAD_W(g1, u1, k_begin + SK_U) }
    const int R = min(*a.pR, a.max_rows);
    if (R <= 0) return;
    const bf16_t *xp = a.X + (size_t)min(lane & 31, R - 1) * a.K + (lane >> 5) * 8;
    SDLM_SK_LOAD_X(x0, k_begin)
    if (k_begin + SK_U < k_end) { SDLM_SK_LOAD_X(x1, k_begin + SK_U) }
    f32x16 ag, au;
#pragma unroll
    for (int v = 0; v < 16; ++v) { ag[v] = 0.f; au[v] = 0.f; }
    for (int k0 = k_begin; k0 < k_end; k0 += 2 * SK_U) {
        SDLM_SK_MMA(g0, u0, x0, k0)
        if (k0 + 2 * SK_U < k_end) { SDLM_SK_LOAD_W(g0, u0, k0 + 2 * SK_U) SDLM_SK_LOAD_X(x0, k0 + 2 * SK_U) }
        SDLM_SK_MMA(g1, u1, x1, k0 + SK_U)
        if (k0 + 3 * SK_U < k_end) { SDLM_SK_LOAD_W(g1, u1, k0 + 3 * SK_U) SDLM_SK_LOAD_X(x1, k0 + 3 * SK_U) }
    }
#undef SDLM_SK_LOAD_W
#undef SDLM_SK_LOAD_X
#undef SDLM_SK_MMA
#pragma unroll
    for (int v = 0; v < 16; ++v) { part[wave][0][v][lane] = ag[v]; part[wave][1][v][lane] = au[v]; }
    __syncthreads();
    // accumulator element v of lane l: feature 8*(v/4) + 4*(l/32) + v%4 of the block, activation row l%32;
    // wavefront w finishes the elements EL*w .. EL*w + EL-1 of every lane: EL consecutive features of one row
    constexpr int EL = 16 / SK_W;
    static_assert(EL == 2 || EL == 4, "an output store is one or two bf16 pairs");
    const int row = lane & 31, v0 = wave * EL, n = j * 32 + (v0 >> 2) * 8 + (lane >> 5) * 4 + (v0 & 3);
    if (row >= R || n >= a.N) return;
    float o[EL];
#pragma unroll
    for (int e = 0; e < EL; ++e) {
        float gs = part[0][0][v0 + e][lane], us = part[0][1][v0 + e][lane];
#pragma unroll
        for (int w = 1; w < SK_W; ++w) { gs += part[w][0][v0 + e][lane]; us += part[w][1][v0 + e][lane]; }
        o[e] = silu_f(gs) * us;
    }
    bf16_t *dst = a.Yt + (size_t)row * a.n_out + n;
    if constexpr (EL == 4) *(uint2 *)dst = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
    else *(uint32_t *)dst = pack_bf16(o[0], o[EL - 1]);
}

// ------------------------------------------------------------------------------------------------ steps of few rows
// The step of a single sequence, or of a few with small blocks, has at most 16 or 32 rows.  Its products are weight streams and
// nothing else, bound by how evenly the stream is dealt out to the compute units and by how much of it is requested at
// once.  They share one inner loop: a workgroup owns two 16-feature tiles, its four wavefronts each take a quarter of its k range,
// and the quarters are added in wavefront order through LDS.  Both operands come straight from global memory in the order of
// v_mfma_f32_16x16x32_bf16: a 16-feature half of a packed 32 x 16 tile pair is four runs of 256 bytes per load, the rows (shared by
// every workgroup, so served by L2) are a run of 1 KB a step where their writer leaves them in operand order (ordered_off: QKV, and gate/up and down of
// the chain below), else 64 pieces of 16 bytes; rows beyond the live ones repeat the last row and their results are dropped.  The order is worth most
// with many rows: a step of the 3B shape, 18 layers, 160 rows 2156 -> 2098 us, 5 rows no difference.  NB = 1 serves at most 16 rows, NB = 2 at most 32 (QKV also takes more rows, in blocks: see qkv_rows).  Against workgroups of 32-feature tiles (the tiled kernel for O and
// down, which also stages the rows in LDS slice by slice), before -> after in a step of 5 / 16 rows (us; what
// is launched where is decided by few16_resid and few16_gateup):
//   h = 1536, F = 8960    QKV 9.4 -> 6.8 / 10.0 -> 7.9,  O 5.5 -> 4.6 / 5.5 -> 5.0, down 9.3 -> 6.9 / 9.6 -> 7.9, gate/up 15.9 -> 14.7 / 17.2 -> 17.3
//   h = 2048, F = 11008   QKV 10.9 -> 7.2 / 12.5 -> 8.0, O 5.6 -> 5.0 / 5.9 -> 5.2, down 12.3 -> 11.3 / 11.9 -> 13.0 (with half the slabs),
//                         gate/up 22.0 -> 19.2 / 23.2 -> 21.7
//   h = 3584, F = 18944   QKV 17.6 -> 12.0 / 18.6 -> 13.3, O 7.9 -> 7.5 / 8.2 -> 8.2 (4 slabs instead of 14), gate/up 53.3 -> 50.9 / 54.6 -> 55.9
//   h = 5120, F = 27648   QKV 25.1 -> 17.1 / 26.9 -> 19.3, O and down 68.1 -> 63.5 / 70.6 -> 70.7 (3 slabs instead of 12 and 13),
//                         gate/up 104.4 -> 101.5 / 108.5 -> 111.4
// With 17 to 32 rows the rows' requests double: QKV, whose 2 x 32-feature workgroups were fewest, still gains (h = 2048 12.9 -> 10.7 us,
// h = 5120 28.4 -> 22.4); gate/up (h = 5120 115 -> 130) and down (h = 3584 27.6 -> 38) lose and keep their kernels.
constexpr int sk_u(int NB) { return NB == 1 ? 8 : NB == 2 ? 6 : 3; }   // k steps (of 32) per register set: two wavefronts per SIMD

// Products of the features whose first elements `wa` and `wb` point to (each the start of a 16-feature half of a packed tile)
// with the 16 NB rows of X from m0 on, over k steps [k_begin, k_end); steps beyond k_end repeat the last one.  `with_rows` runs after
// the row count is known and the first operands are requested: the caller's own requests go there.  Returns the row count.
// Result: element v of lane l is feature 4 * (l / 16) + v of the tile, row m0 + 16 * nb + l % 16.
template <int NB, int NT, bool XP, int U, class F>
__device__ inline int skinny_dot(const bf16_t *wa, const bf16_t *wb, const bf16_t *X, const int32_t *pR, int max_rows, int m0, int K, int k_begin, int k_end,
                                 int lane, f32x4 (&aa)[NB], f32x4 (&ab)[NB], F with_rows)
{
    const int k_last = max(k_end, 1) - 1;   // a wavefront without any k step still requests within the matrix
    // lane -> k half of the step's 32 (lane / 32), 8 of 16 (lane / 16 % 2), feature (lane % 16)
    const uint32_t wl = (lane >> 5) * 512 + ((lane & 15) + ((lane >> 4) & 1) * 32) * 8;
    bf16x8 a0[U], b0[U], x0[NB][U], a1[U], b1[U], x1[NB][U];
    const bf16_t *xp[NB];
    auto load_w = [&](bf16x8 (&A)[U], bf16x8 (&B)[U], int k) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t o = (size_t)min(k + u, k_last) * 1024;
            A[u] = *(const bf16x8 *)(wa + o + wl);
            if constexpr (NT == 2) B[u] = *(const bf16x8 *)(wb + o + wl);
        }
    };
    auto load_x = [&](bf16x8 (&Xr)[NB][U], int k) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) Xr[nb][u] = *(const bf16x8 *)(xp[nb] + min(k + u, k_last) * (XP ? 512 : 32));
    };
    auto mma = [&](const bf16x8 (&A)[U], const bf16x8 (&B)[U], const bf16x8 (&Xr)[NB][U], int k) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k + u < k_end) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    aa[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[u], Xr[nb][u], aa[nb], 0, 0, 0);
                    if constexpr (NT == 2) ab[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(B[u], Xr[nb][u], ab[nb], 0, 0, 0);
                }
            }
    };
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) { aa[nb] = f32x4{0.f, 0.f, 0.f, 0.f}; ab[nb] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    load_w(a0, b0, k_begin);   // the weights do not wait for the row count
    if (k_begin + U < k_end) load_w(a1, b1, k_begin + U);
    const int R = min(*pR, max_rows);
    if (R <= m0) return 0;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int r = min(m0 + nb * 16 + (lane & 15), R - 1);
        xp[nb] = X + (XP ? ordered_off(r, (lane >> 4) * 8, K) : (size_t)r * K + (lane >> 4) * 8);
    }
    load_x(x0, k_begin);
    if (k_begin + U < k_end) load_x(x1, k_begin + U);
    with_rows(R);
    for (int k = k_begin; k < k_end; k += 2 * U) {
        mma(a0, b0, x0, k);
        if (k + 2 * U < k_end) { load_w(a0, b0, k + 2 * U); load_x(x0, k + 2 * U); }
        mma(a1, b1, x1, k + U);
        if (k + 3 * U < k_end) { load_w(a1, b1, k + 3 * U); load_x(x1, k + 3 * U); }
    }
    return R;
}

// The four quarters of k, added in wavefront order.  Wavefront nb < NB finishes rows 16 nb .. 16 nb + 15; the others return false.
template <int NB>
__device__ inline bool skinny_sum(f32x4 (&part)[SK_W][2][NB][64], const f32x4 (&aa)[NB], const f32x4 (&ab)[NB], int wave, int lane, f32x4 &sa, f32x4 &sb)
{
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) { part[wave][0][nb][lane] = aa[nb]; part[wave][1][nb][lane] = ab[nb]; }
    __syncthreads();
    if (wave >= NB) return false;
    sa = part[0][0][wave][lane]; sb = part[0][1][wave][lane];
#pragma unroll
    for (int w = 1; w < SK_W; ++w) { sa += part[w][0][wave][lane]; sb += part[w][1][wave][lane]; }
    return true;
}

// ---- norms inside the products: the chain of a step of at most 16 rows (launch_*_few below)
// Such a step is a chain of launches, and the two RMSNorms of a layer, with the split-k slabs that they add, were two of eight.  Here O and down sum all of k
// inside a workgroup of 16 features, so that its epilogue has the finished residual stream: it stores x, x times the gains of the norm that follows (bf16, the operand
// of the next product), and the sum of squares of its 16 features per row.  The next product multiplies its sums by 1 / rms, from those h / 16 sums of squares, which
// it requests first and adds while its weights are under way.  x g is rounded to bf16 before the factor 1 / rms instead of behind it: the same relative rounding.
// The operands are kept in the order of the matrix instruction, [k / 32][k / 8 % 4][row][8], so that a load is one run of up to 1 KB and not 64 pieces
// of 16 bytes; gate/up leaves its result in that order too.  Whole steps of one sequence of 512 tokens, D = 4, us: h = 1536, F = 8960, 28 layers 1613 -> 1513, h = 2048, F = 11008, 18 layers
// 1279 -> 1215, h = 3584, F = 18944, 8 layers 1209 -> 1138 (16 rows 1259 -> 1186), h = 5120, F = 27648, 8 layers 1976 -> 1965.
constexpr int FEW_SSQ = 8;   // requests of 16 bytes a lane: h up to 8192

struct FewRms {
    float4 v[FEW_SSQ];
    // wavefront w of SK_W takes every SK_W-th run of 16 sums of its rows; row = lane % 16
    __device__ void request(const float *ssq, int n, int wave, int lane)
    {
#pragma unroll
        for (int t = 0; t < FEW_SSQ; ++t) {
            const int i = ((t * SK_W + wave) * 4 + (lane >> 4)) * 4;
            v[t] = i < n ? *(const float4 *)(ssq + (size_t)(lane & 15) * n + i) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
    __device__ void add(float (&rs)[SK_W][16], int wave, int lane) const
    {
        float s = 0.f;
#pragma unroll
        for (int t = 0; t < FEW_SSQ; ++t) s += (v[t].x + v[t].y) + (v[t].z + v[t].w);
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (lane < 16) rs[wave][lane] = s;
    }
    // behind a barrier
    static __device__ float factor(const float (&rs)[SK_W][16], int row, int h, float eps)
    {
        float s = rs[0][row];
#pragma unroll
        for (int w = 1; w < SK_W; ++w) s += rs[w][row];
        return 1.0f / sqrtf(s / (float)h + eps);
    }
};

// Gate/up: SiLU(gate) * up needs complete sums, so k cannot be split between workgroups; a workgroup owns 16 features.
// NORM: rows and result in operand order, the norm's factor here.
template <bool NORM>
__global__ __launch_bounds__(SK_W * 64) void swiglu_skinny16_k(MfmaArgs a)
{
    constexpr int NB = 1;
    __shared__ f32x4 part[SK_W][2][NB][64];
    __shared__ float rs[SK_W][16];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = blockIdx.x >> 1, h = blockIdx.x & 1;   // features 32 j + 16 h ..: halves of tiles 2j (gate) and 2j + 1 (up) of the fused matrix
    const int KS = a.K >> 4, K32 = a.K >> 5, per = (K32 + SK_W - 1) / SK_W;
    const bf16_t *wg = a.Wp + ((size_t)(2 * j) * KS) * 512 + h * 128;
    f32x4 ag[NB], au[NB], gs, us;
    FewRms rms;
    if constexpr (NORM) rms.request(a.ssq, a.K >> 4, wave, lane);
    const int R = skinny_dot<NB, 2, NORM, sk_u(NB)>(wg, wg + (size_t)KS * 512, a.X, a.pR, a.max_rows, 0, a.K, wave * per, min(K32, wave * per + per), lane, ag, au,
                                                    [&](int) { if constexpr (NORM) rms.add(rs, wave, lane); });
    if (R <= 0 || !skinny_sum<NB>(part, ag, au, wave, lane, gs, us)) return;
    const int row = wave * 16 + (lane & 15), n = j * 32 + h * 16 + (lane >> 4) * 4;
    if (row >= R || n >= a.N) return;
    if constexpr (NORM) {
        const float f = FewRms::factor(rs, row, a.K, a.eps);
        gs *= f;
        us *= f;
    }
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = silu_f(gs[e]) * us[e];
    *(uint2 *)(a.Yt + (NORM ? ordered_off(row, n, a.N) : (size_t)row * a.n_out + n)) = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
}

// O of that chain, and down where few_down_whole says so: all of k by the eight wavefronts of a workgroup of 16 NT features.  XP: rows in operand order (down).
// Bound: the operands' requests of one workgroup, weights and rows alike 1 KB a k step, which a compute unit serves at 75 GB/s; four k steps a register set (four
// wavefronts a SIMD) are as fast as six, 16 wavefronts or 32 features a workgroup slower (h = 1536, F = 8960, 8 rows, whole step 1502 us; six k steps 1504, 16
// wavefronts 1518, 32 features 1652).  O with its norm, h = 1536, 5 rows: 9.1 us in two launches, now 5.2.
constexpr int FEW_W = 8, FEW_U = 4;

template <bool XP, int NT>
__global__ __launch_bounds__(FEW_W * 64) void resid_few_k(MfmaArgs a)
{
    __shared__ f32x4 part[FEW_W][NT][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t16 = blockIdx.x * NT, n = (t16 + (NT == 2 ? wave & 1 : 0)) * 16 + (lane >> 4) * 4, row = lane & 15, K32 = a.K >> 5;
    const bf16_t *w = a.Wp + (size_t)(t16 >> 1) * (a.K >> 4) * 512 + (t16 & 1) * 128;
    const int kb = (int)((long)K32 * wave / FEW_W), ke = (int)((long)K32 * (wave + 1) / FEW_W);
    f32x4 aa[1], ab[1], x;
    uint2 g = make_uint2(0, 0);
    const int R = skinny_dot<1, NT, XP, FEW_U>(w, w + 128, a.X, a.pR, a.max_rows, 0, a.K, kb, ke, lane, aa, ab, [&](int rows) {
        if (wave >= NT) return;
        x = *(const f32x4 *)(a.Yf + (size_t)min(row, rows - 1) * a.n_out + n);
        if (a.gain) g = *(const uint2 *)(a.gain + n);
    });
    if (R <= 0) return;
    part[wave][0][lane] = aa[0];
    if constexpr (NT == 2) part[wave][1][lane] = ab[0];
    __syncthreads();
    if (wave >= NT) return;   // wavefront i finishes the features of tile i
    f32x4 s = part[0][wave][lane];
#pragma unroll
    for (int i = 1; i < FEW_W; ++i) s += part[i][wave][lane];
    x += s;
    if (row < R) *(f32x4 *)(a.Yf + (size_t)row * a.n_out + n) = x;
    if (!a.gain) return;   // behind the last layer
    float ss = (x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]);
    ss += __shfl_xor(ss, 16);
    ss += __shfl_xor(ss, 32);
    if (row >= R) return;
    if (lane < 16) a.ssq[(size_t)row * (a.n_out >> 4) + t16 + wave] = ss;
    const float g0 = bf16_to_f((bf16_t)(g.x & 0xffff)), g1 = bf16_to_f((bf16_t)(g.x >> 16)), g2 = bf16_to_f((bf16_t)(g.y & 0xffff)), g3 = bf16_to_f((bf16_t)(g.y >> 16));
    *(uint2 *)(a.xg + ordered_off(row, n, a.n_out)) = make_uint2(pack_bf16(x[0] * g0, x[1] * g1), pack_bf16(x[2] * g2, x[3] * g3));
}

// The embeddings of that chain's rows, in the same three forms.  Four features a thread.
__global__ __launch_bounds__(256) void embed_few_k(float *x, const bf16_t *E, const int32_t *tok, const int32_t *pR, int h, int V, const bf16_t *gain, bf16_t *xg, float *ssq)
{
    const int r = blockIdx.y, n = (blockIdx.x * 256 + threadIdx.x) * 4;   // h is a multiple of 64: the four lanes of 16 features are all there or none
    if (r >= *pR || n >= h) return;
    const uint2 e = *(const uint2 *)(E + (size_t)min(max(tok[r], 0), V - 1) * h + n), g = *(const uint2 *)(gain + n);
    const float4 v = make_float4(bf16_to_f((bf16_t)(e.x & 0xffff)), bf16_to_f((bf16_t)(e.x >> 16)), bf16_to_f((bf16_t)(e.y & 0xffff)), bf16_to_f((bf16_t)(e.y >> 16)));
    *(float4 *)(x + (size_t)r * h + n) = v;
    *(uint2 *)(xg + ordered_off(r, n, h)) = make_uint2(pack_bf16(v.x * bf16_to_f((bf16_t)(g.x & 0xffff)), v.y * bf16_to_f((bf16_t)(g.x >> 16))),
                                                pack_bf16(v.z * bf16_to_f((bf16_t)(g.y & 0xffff)), v.w * bf16_to_f((bf16_t)(g.y >> 16))));
    float ss = (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
    ss += __shfl_xor(ss, 1);
    ss += __shfl_xor(ss, 2);
    if ((threadIdx.x & 3) == 0) ssq[(size_t)r * (h >> 4) + (n >> 4)] = ss;
}

// O and down projection: a workgroup owns a packed tile's 32 features and one of `splits` ranges of k; slabs as in the tiled kernel.  XP: rows in operand order.
template <bool XP>
__global__ __launch_bounds__(SK_W * 64) void resid_skinny_k(MfmaArgs a)
{
    constexpr int NB = 1;
    __shared__ f32x4 part[SK_W][2][NB][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.x / a.splits, split = blockIdx.x % a.splits;
    const int K32 = a.K >> 5, k0 = (int)((long)K32 * split / a.splits), k1 = (int)((long)K32 * (split + 1) / a.splits), per = (k1 - k0 + SK_W - 1) / SK_W;
    const int kb = min(k1, k0 + wave * per);
    const bf16_t *w = a.Wp + (size_t)tile * (a.K >> 4) * 512;
    f32x4 aa[NB], ab[NB], s[2];
    const int R = skinny_dot<NB, 2, XP, sk_u(NB)>(w, w + 128, a.X, a.pR, a.max_rows, 0, a.K, kb, min(k1, kb + per), lane, aa, ab, [](int) {});
    if (R <= 0 || !skinny_sum<NB>(part, aa, ab, wave, lane, s[0], s[1])) return;
    const int row = wave * 16 + (lane & 15);
    if (row >= R) return;
    float *dst = a.Yf + (a.splits > 1 ? (size_t)split * a.slab : 0) + (size_t)row * a.n_out + tile * 32 + (lane >> 4) * 4;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        f32x4 *p = (f32x4 *)(dst + t * 16);
        if (a.splits > 1) *p = s[t]; else *p += s[t];
    }
}

// QKV projection, rotation and K/V placement in one kernel: such steps are bound by their kernel boundaries, and here the
// projection needs no split along k between workgroups, so its epilogue sees complete sums.  A workgroup owns features
// [16 t, 16 t + 16) and the same range 64 further on of one head, i.e. both members of every rotate-half pair (i, i + d/2).  The
// epilogue is the RoPE + K/V placement kernel's: queries and keys rotated at the row's position, a pending row's K/V to the cache
// slot of its position, any other row's to slot `kind` of its staging tile.
struct QkvSkinnyArgs {
    const bf16_t *X, *Wp, *bias;
    const int32_t *pR;
    int max_rows, K, Hq;
    int m_sure, m_rest;     // row blocks that certainly hold rows, and that may
    bf16_t *q_out, *pool;
    KvGeom kg;
    RowMeta rm;
    SeqState st;
    const float2 *rope;
    const float *ssq;       // NORM: X is x times the gains in operand order
    float eps;
};

// The 16 NB rows from m0 on, columns `col`.
template <int NB, bool NORM>
__device__ inline void qkv_rope_rows(const QkvSkinnyArgs &a, f32x4 (&part)[SK_W][2][NB][64], int m0, int col, int lane, int wave)
{
    const int head = col >> 2, t16 = col & 3;   // heads: Hq of q, then Hkv of k, then Hkv of v; t16: which 16 of the first 64 features
    const int KS = a.K >> 4, K32 = a.K >> 5, per = (K32 + SK_W - 1) / SK_W;
    const bf16_t *wa = a.Wp + ((size_t)(head * 4 + (t16 >> 1)) * KS) * 512 + (t16 & 1) * 128;
    const int d = a.kg.head_dim, half = d >> 1, Hk = a.kg.n_kv_heads;
    const int i0 = t16 * 16 + (lane >> 4) * 4;   // this lane's four features: index within the first half of the head
    const bool is_q = head < a.Hq, is_v = head >= a.Hq + Hk;
    const int row = m0 + wave * 16 + (lane & 15);
    float2 t[4];
    float blo[4] = {0.f, 0.f, 0.f, 0.f}, bhi[4] = {0.f, 0.f, 0.f, 0.f};
    int page = -1, slot = 0;
    f32x4 aa[NB], ab[NB], sa, sb;
    __shared__ float rs[NORM ? SK_W : 1][16];
    FewRms rms;
    if constexpr (NORM) rms.request(a.ssq, a.K >> 4, wave, lane);
    // what the epilogue needs beside the sums is requested with the operands: rotation factors, bias, the page of a cached position
    const int R = skinny_dot<NB, 2, true, sk_u(NB)>(wa, wa + (size_t)2 * KS * 512, a.X, a.pR, a.max_rows, m0, a.K, wave * per, min(K32, wave * per + per), lane, aa, ab, [&](int rows) {
        if constexpr (NORM) rms.add(rs, wave, lane);
        if (wave >= NB) return;
        const int rr = min(row, rows - 1), pos = a.rm.pos[rr], kind = a.rm.kind[rr], b = a.rm.seq[rr], stg = a.rm.stg[rr];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            t[e] = is_v ? make_float2(1.f, 0.f) : a.rope[(size_t)pos * half + i0 + e];
            if (a.bias) { blo[e] = bf16_to_f(a.bias[head * d + i0 + e]); bhi[e] = bf16_to_f(a.bias[head * d + half + i0 + e]); }
        }
        page = stg; slot = kind;
        if (!is_q && kind < 0) { page = a.st.page_table[(size_t)b * a.kg.pages_per_seq + pos / PAGE]; slot = pos % PAGE; }
    });
    if (R <= 0 || !skinny_sum<NB>(part, aa, ab, wave, lane, sa, sb) || row >= R) return;
    if constexpr (NORM) {
        const float f = FewRms::factor(rs, row, a.K, a.eps);
        sa *= f;
        sb *= f;
    }
    float lo[4], hi[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float va = sa[e] + blo[e], vb = sb[e] + bhi[e];
        lo[e] = is_v ? va : va * t[e].x - vb * t[e].y;
        hi[e] = is_v ? vb : vb * t[e].x + va * t[e].y;
    }
    if (is_q) {
        bf16_t *q = a.q_out + ((size_t)row * a.Hq + head) * d + i0;
        *(uint2 *)q = make_uint2(pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]));
        *(uint2 *)(q + half) = make_uint2(pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3]));
        return;
    }
    if (page < 0) return;   // unbacked position: only reachable after a reported pool exhaustion
    const int hk = is_v ? head - a.Hq - Hk : head - a.Hq;
    bf16_t *tile = a.pool + a.kg.tile(page, hk);
    if (!is_v) {
        // k_off(slot, i) keeps eight consecutive features of a slot together: i0 is a multiple of four
        *(uint2 *)(tile + k_off(slot, i0)) = make_uint2(pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]));
        *(uint2 *)(tile + k_off(slot, i0 + half)) = make_uint2(pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3]));
    } else {
        bf16_t *Vb = tile + PAGE * d;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            Vb[v_off(slot, i0 + e)] = f_to_bf16(lo[e]);
            Vb[v_off(slot, i0 + half + e)] = f_to_bf16(hi[e]);
        }
    }
}

// Row blocks of 16 NB rows; those that may be empty are of 16 NR rows.
template <int NB, int NR, bool NORM = false>
__global__ __launch_bounds__(SK_W * 64, 2) void qkv_rope_skinny_k(QkvSkinnyArgs a)
{
    __shared__ f32x4 part[SK_W * 2 * NB * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroup id -> (row block, column block), as in the tiled kernel: certain row blocks first, the row blocks of one
    // column block on one XCD, so that its weights leave memory once
    const int n_cols = 4 * (a.Hq + 2 * a.kg.n_kv_heads), n_first = n_cols * a.m_sure, first8 = (n_first + 7) & ~7;
    const bool sure = (int)blockIdx.x < first8;
    const int bid = sure ? blockIdx.x : blockIdx.x - first8, mb = sure ? a.m_sure : a.m_rest;
    const int per8 = (n_cols * mb + 7) >> 3, wg = (bid & 7) * per8 + (bid >> 3);
    if (wg >= n_cols * mb) return;
    const int m0 = NB == NR ? ((sure ? 0 : a.m_sure) + wg % mb) * NB * 16 : (sure ? 0 : a.m_sure * NB * 16) + wg % mb * (sure ? NB : NR) * 16;
    if (!sure && m0 >= *a.pR) return;
    // (one copy of the body where one will do, and the block's first row as one product: 0.2 us of a launch of 6.6)
    if (NB == NR || sure) qkv_rope_rows<NB, NORM>(a, *reinterpret_cast<f32x4 (*)[SK_W][2][NB][64]>(part), m0, wg / mb, lane, wave);
    else qkv_rope_rows<NR, false>(a, *reinterpret_cast<f32x4 (*)[SK_W][2][NR][64]>(part), m0, wg / mb, lane, wave);
}

static int sure_blocks(int rows, int min_rows, int MT)
{
    const int mb = (rows + MT * 32 - 1) / (MT * 32);
    if (min_rows <= 0) return mb;
    const int ms = (min_rows + MT * 32 - 1) / (MT * 32);
    return ms < 1 ? 1 : (ms > mb ? mb : ms);
}

// How the fused launch deals out its rows; units = 0: the tiled projection and the RoPE + K/V placement kernel serve this step better.
// Row blocks repeat the weight stream (from L2) and a workgroup's time grows with k times its rows, where the tiled kernel splits
// k between workgroups: row blocks pay while all workgroups fit the chip at once (about one per compute unit).
//   32-row blocks, counted for the mean of certain and possible rows: h = 2048, 66 rows, 240 workgroups 15.1 -> 10.5 us (both kernels
//   before -> fused); h = 1536, 60 rows 13.6 -> 8.9; h = 3584, 432 workgroups slower still (24 sequences, D = 4, a step of 8 layers 1733 -> 1772).
//   64-row blocks, with the rows in operand order, in rounds of two workgroups a unit: k of at most 1536 until the certain rows are a little more than one round of them, four layers of a
//   pass of h = 1536, us: 200 rows 417 -> 383, 320 rows 448 -> 417, 509 rows (512 workgroups) 546 -> 518, 640 rows (640) 596 -> 589, 800 rows 648 -> 647; steps of 14 layers, 64 sequences, D = 4
//   1700 -> 1590, 40 sequences, D = 8 1795 -> 1723.  k of at most 2048 until 400: h = 2048, 320 rows 526 -> 508, 400 rows (560) 572 -> 577, 509 rows 644 -> 656; steps of 18 layers, 40 sequences, D = 4
//   2290 -> 2230.  Longer k: h = 3584, 200 rows 769 -> 800.  The two lines are those of the two widths measured first; between them, over 159 shapes of k = 512 to 2048 with exact rows, one launch
//   is 2 to 9 us a layer ahead wherever it is taken, and where it is not, still ahead by 1 to 6 us up to about 800 workgroups (k of at most 1280 to 1600) and 640 (1600, 1792), behind beyond 1000.
// Blocks that may be empty are of 32 rows, unless all blocks are on the chip at once anyway: a step's rows end in one of them, and a second 64-row workgroup on
// some units would make the launch wait (64 sequences, D = 2, h = 2048, 10 layers 1256 us with 64 rows, 1246 with 32; 64 sequences, D = 4 1761, 1745).  With
// 32 rows where they do fit, a layer takes 3 % longer (24 sequences, D = 4, 192 rows: 114.2 -> 118.2 us).
struct QkvRows { int units, rest_units, m_sure, m_rest; };   // 16-row units of a certain row block and of one that may be empty; how many of each

static QkvRows qkv_rows(const sdlm_model_cfg *m, int max_rows, int min_rows)
{
    if (!mfma_supported(m)) return {};
    const int cols = 4 * (m->n_q_heads + 2 * m->n_kv_heads), chip = 256;
    auto with = [&](int units, int rest_units) {
        const int rows = 16 * units, rest = 16 * rest_units, all = (max_rows + rows - 1) / rows;
        const int m_sure = min(max((min_rows + rows - 1) / rows, 1), all);
        return QkvRows{units, rest_units, m_sure, max(0, (max_rows - m_sure * rows + rest - 1) / rest)};
    };
    if (max_rows <= 16) return with(1, 1);
    if (max_rows <= 32) return with(2, 2);
    if (cols * (sure_blocks(max_rows, min_rows, 1) + (max_rows + 31) / 32) <= 2 * chip) return with(2, 2);
    const int sure = cols * sure_blocks(max_rows, min_rows, 2), all = cols * ((max_rows + 63) / 64);
    if (m->hidden > 2048 || sure > (m->hidden <= 1536 ? 576 : 400)) return {};
    return all <= chip || all == sure ? with(4, 4) : with(4, 2);
}

void mfma_qkv_rows(const sdlm_model_cfg *m, int max_rows, int min_rows, int *rows, int *rest_rows)
{
    const QkvRows q = qkv_rows(m, max_rows, min_rows);
    *rows = 16 * q.units;
    *rest_rows = 16 * q.rest_units;
}

bool qkv_rope_skinny_applies(const sdlm_model_cfg *m, int max_rows, int min_rows) { return qkv_rows(m, max_rows, min_rows).units > 0; }

void launch_qkv_rope_skinny(hipStream_t s, const sdlm_model_cfg *m, const void *X, const void *w_packed, const void *bias, const int32_t *p_rows,
                            int max_rows, int min_rows, void *q_out, void *pool_layer, const KvGeom &kg, const RowMeta &rm, const SeqState &st, const float2 *rope,
                            const float *ssq, float eps)
{
    const QkvRows q = qkv_rows(m, max_rows, min_rows);
    QkvSkinnyArgs a;
    a.X = (const bf16_t *)X; a.Wp = (const bf16_t *)w_packed; a.bias = (const bf16_t *)bias; a.pR = p_rows;
    a.max_rows = max_rows; a.K = m->hidden; a.Hq = m->n_q_heads;
    a.m_sure = q.m_sure; a.m_rest = q.m_rest;
    a.q_out = (bf16_t *)q_out; a.pool = (bf16_t *)pool_layer; a.kg = kg; a.rm = rm; a.st = st; a.rope = rope; a.ssq = ssq; a.eps = eps;
    const int n_cols = 4 * (m->n_q_heads + 2 * m->n_kv_heads);
    const dim3 grid((n_cols * a.m_sure + 7) / 8 * 8 + (n_cols * a.m_rest + 7) / 8 * 8), block(SK_W * 64);
    if (ssq) hipLaunchKernelGGL((qkv_rope_skinny_k<1, 1, true>), grid, block, 0, s, a);
    else if (q.units == 1) hipLaunchKernelGGL((qkv_rope_skinny_k<1, 1>), grid, block, 0, s, a);
    else if (q.units == 2) hipLaunchKernelGGL((qkv_rope_skinny_k<2, 2>), grid, block, 0, s, a);
    else if (q.rest_units == 4) hipLaunchKernelGGL((qkv_rope_skinny_k<4, 4>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((qkv_rope_skinny_k<4, 2>), grid, block, 0, s, a);
}

// ------------------------------------------------------------------------------------------------ launch policy
// k splits of an O or down projection in the stream for at most 16 rows: at most two workgroups per compute unit, so that all run at
// once (h = 1536, F = 8960: 11 splits, 528 workgroups 8.9 us, 10 splits 7.2 us), and at least 512 of k each.
static int skinny_splits(int rows, int N, int K, size_t slab_room_floats)
{
    long sp = 512 / (long)(mfma_pad_n(N) / 32);
    const long cap_k = K / 512, cap_m = (long)(slab_room_floats / ((size_t)rows * N));
    sp = sp > cap_k ? cap_k : sp;
    sp = sp > cap_m ? cap_m : sp;
    sp = sp > 16 ? 16 : sp;
    return (int)(sp < 1 ? 1 : sp);
}

// Whether an O or down projection of at most 16 rows runs as that stream, or as the tiled kernel.  Up to k = 6144 the stream has the shorter
// launch by 5 to 35 %, whatever the rows (us with the RMSNorm that adds the slabs, tiled -> stream: N = K = 1536 7.9 -> 7.5, 3584 14.2 -> 12.2,
// 5120 18.6 -> 18.5, all at 16 rows, and more at fewer).  With longer k the rows' requests, which the stream repeats in every workgroup,
// begin to weigh, and two things turn it:
//   * workgroups that are neither one round of the units nor (nearly) two: N = 3584, K = 18944, 448 workgroups: 5 rows 30.8 -> 30.6, 8 rows 31.1 -> 31.9,
//     16 rows 31.9 -> 35.5; N = 6144, K = 16384, 384: 5 rows 46.6 -> 47.5, 16 rows 48.5 -> 52.7;
//   * more than 12 rows, where the tiled kernel's own workgroups are one to two rounds: N = 4096, K = 14336: 8 rows 28.4 -> 28.2, 16 rows 29.2 -> 30.4;
//     N = 2048, K = 11008: 10 rows 16.7 -> 16.0, 16 rows 16.9 -> 17.1.  Elsewhere the stream keeps its lead: N = 1536, K = 8960 (192 tiled
//     workgroups) 16 rows 14.5 -> 12.5, N = 5120, K = 27648 (520) 62.1 -> 58.8.
static bool few16_resid(int min_rows, int N, int K, int splits)
{
    if (K <= 6144) return true;
    const long wgs = (long)(N / 32) * splits, blocks = (N + 127) / 128, tiled = blocks * min(16L, (512 + blocks - 1) / blocks);
    return !(wgs > 256 && wgs < 480) && !(min_rows > 12 && tiled >= 256 && tiled <= 512);
}

// Whether gate/up of at most 16 rows runs in 16-feature blocks, or in the 32-feature blocks that serve up to 32 rows.  The finer blocks spread
// the stream better over the units (us, 32 -> 16 features, at 5 / 16 rows: N = 8960, K = 1536 15.5 -> 14.2 / 16.8 -> 16.7; N = 11008, K = 2048 21.7 -> 17.8 /
// 22.7 -> 20.5; N = 18944, K = 3584 52.0 -> 49.6 / 54.9 -> 56.3; N = 27648, K = 5120 99.9 -> 97.6 / 104.7 -> 106.7), but repeat the rows' requests
// twice as often.  The coarser ones win where they are one round of the units themselves (N = 6912, K = 2560, 216 blocks: 15.3 -> 16.0 / 15.8 -> 18.6;
// N = 8192, K = 3072, 256: 19.9 -> 19.2 / 20.4 -> 21.7), and with more than 12 rows where they are more than two.
static bool few16_gateup(int min_rows, int N)
{
    const int blocks32 = (N + 31) / 32;
    return !(blocks32 >= 144 && blocks32 <= 256 && min_rows > 4) && !(blocks32 > 512 && min_rows > 12);
}

// (Both rules are those of passes with separate norms: prompts of at most 16 tokens, widths above 8192.  In the chain of a decode step the operands' order makes the finer
// gate/up blocks and the stream of down better than what these rules choose: h = 5120, F = 27648, 16 rows, a step of 8 layers 1973 -> 1944 us; 144 to 256 blocks of 32 features, whole steps of six
// layers before the chain / with it: h = 2560, F = 6912, 6 rows 434 / 410, 12 rows 444 / 416, 16 rows 468 / 428, h = 3072, F = 8192, 12 rows 519 / 473, h = 4096, F = 8192 634 / 559.)
// What a product runs as: FEW16 / FEW32 are the kernels without LDS tiles for steps of few rows (16 rows x two 16-feature tiles, 32 rows x two
// 32-feature tiles a workgroup), TILED the tiled kernel.
enum { TILED = 0, FEW16, FEW32 };
struct TileChoice { int kind, MT, NT, splits, WV, KH; };

// Gate/up launches of more than 32 rows whose shape the plain tiles do not serve well (K a multiple of 128):
//   * Up to 128 possible rows and at most 256 column blocks of 64 features: workgroups of 64 or 128 rows x 64 features whose wavefronts
//     take half of k each.  Bound by the weights in flight: F / 128 workgroups of the plain tile leave most compute units without any (h = 2048,
//     F = 11008: 86 workgroups); half the columns double the workgroups, and k in halves keeps four wavefronts in each.
//     h = 2048, F = 11008: 66 rows 32.9 -> 24.4 us, 48 rows 35.6 -> 24.8; h = 1536, F = 8960: 96 rows 24.5 -> 19.7, 48 rows 27.4 ->
//     18.9; h = 4096, F = 16384 (256 blocks): 48 rows 70.9 -> 52.4, 128 rows 66.9 -> 56.7.  A workgroup of 128 rows fills a unit (360 registers), so
//     beyond 256 blocks there is a second round: h = 3584, F = 18944 (296): 70 rows 55.6 -> 70.5; h = 5120, F = 27648 (432): 96 rows 99.4 -> 112.7; those of
//     64 rows are two a unit (48 rows 65.2 and 104.0, the plain 128-row tile 53.0 and 95.1).  With up to 64 possible rows the 128-row workgroup takes over
//     above 40 certain ones (64 rows, h = 2048 24.7 -> 22.4, h = 1536 18.0 -> 16.5; both are equal up to 32 live rows).  Beyond 128 rows (192- and 256-row tiles in halves: 160 rows 31.8 -> 32.5) and for the split-k
//     projections (160 rows, QKV 11.8 -> 19.4, O 8.8 -> 14.0, down 20.8 -> 23.4) the activations' share of the load path takes it back.
//   * Where the 192-row tile would be taken (129 to 192 certain rows) and more than 192 are possible: a 256-row tile, so that the rows from 193 to 256
//     are not a second row block that streams every weight again.  A layer of h = 5120, F = 27648: 208 rows 406 -> 337 us, 256 rows 431 -> 361; up to
//     192 rows it costs 0.8 (315.8 -> 316.6 at 156), and beyond 256, where both need a second block, 6 (20 sequences, D = 8, 320 rows: 423 -> 429).  (Its
//     256 accumulator registers leave room for the operands only with an even number of slices, without a peeled last one.)
static void refine_gateup(int rows, int min_rows, int N, int K, TileChoice *c)
{
    if (K % 128) return;
    if (rows > 32 && rows <= 128 && (N + 63) / 64 <= 256) { c->KH = 2; c->MT = rows <= 64 && min_rows <= 40 ? 2 : 4; c->NT = 2; c->WV = 4; }
    else if (c->MT == 6 && rows > 192) c->MT = 8;
}

// Estimate, in us, of a plain-store or residual product in 128-row tiles of 128 NT columns with `sp` k splits, and of the consumer's reading of the splits'
// slabs.  Fitted to whole steps with every tile and split count of 716 products (N = 512 to 10240, K = 320 to 32512, 34 to 2000 rows): a 64-deep slice takes 0.53 us with 128
// columns and 0.97 with 256, whatever rows of the tile are live, and between 200 and 500 rows, where ever more of the weights are shared and the matrix pipes begin to bound, up to
// 0.70 and 1.07; workgroups of one compute unit share its load path, a second one costs 1.4 times its own slices, later ones 1.5; weights come at 6.4 TB/s where nothing else
// bounds; a megabyte of slabs is written and read in 0.42 us.  Its choice is 0.36 us from the best on average; as many workgroups of the wide tile as units wherever that fits 1.82; with
// the slices' cost as a step at 400 rows and no more than its own slices for a second workgroup it was 0.54, and slower than that rule by up to 16 us.  us a step saved against that over four
// layers, (columns, splits): N = 3840, K = 3072, 409 rows (256, 4) -> (128, 2) 16;  N = 6144, K = 24576, 274 rows (256, 7) -> (256, 3) 115.
// Over 1072 products of 390 other models (h = 1024 to 6144, 34 to 900 rows, many just beyond a multiple of 128) a step is 0.8 % faster than with as many workgroups as units on average, by
// more than 2 % slower in 25 and by 6.9 % at worst (N = 4352, K = 19072, 756 rows, four layers 2402 -> 2567 us).  Blocks of few rows counted by their 32-row tiles, the mean of the costs at certain
// and at likely rows, and the old choice wherever the estimates are close choose no better over those.
// us a launch, (columns, splits) as many as units -> now:
// N = 2048, K = 11008, 160 rows (256, 16) 20.0 -> (128, 8) 18.0;  N = 3584, K = 18944, 49 rows (256, 16) 28.7 -> (128, 9) 27.1;  N = 5120 square,
// 160 rows (256, 6) 20.3 -> (128, 3) 19.7, the norm behind each 0.6 to 2 us shorter;  N = 5120, K = 27648, 992 rows (128, 1) 386 -> (256, 3) 261.
static float tiled_us(int NT, int sp, int rows, int N, int K)
{
    const int S = K / 64, per = (S + sp - 1) / sp;
    const long wgs = (long)((N + 128 * NT - 1) / (128 * NT)) * ((rows + 127) / 128) * sp, rounds = (wgs + 255) / 256;
    const float shared = fminf(1.f, fmaxf(0.f, (rows - 200) / 300.f));
    const float slice = NT == 1 ? 0.53f + 0.17f * shared : 0.97f + 0.10f * shared;
    const float loop = per * slice * (rounds > 1 ? 2.4f + 1.5f * (rounds - 2) : 1.f), weights = (float)N * K * 2 / 6.45e6f;
    const float l2 = loop * loop, w2 = weights * weights;
    const float slabs = sp > 1 ? (float)sp * rows * N * 4 * 0.42e-6f : 0.f;
    return sqrtf(sqrtf(l2 * l2 + w2 * w2)) + slabs;
}

// rows: bound of the launch (grid); min_rows: rows that are certainly there.  The one place where a launch shape is decided.
static TileChoice choose(int epi, int rows, int min_rows, int N, int K, size_t slab_room_floats)
{
    if (epi == EPI_SWIGLU && rows <= 32) return {rows <= 16 && few16_gateup(min_rows, N) ? FEW16 : FEW32, 1, 2, 1, SK_W, SK_W};
    if (epi == EPI_RESID && rows <= 16) {
        const int sp = skinny_splits(rows, N, K, slab_room_floats);
        if (few16_resid(min_rows, N, K, sp)) return {FEW16, 1, 1, sp, SK_W, SK_W};
    }
    TileChoice c{TILED, rows <= 32 ? 1 : rows <= 64 ? 2 : 4, 2, 1, 4, 1};
    // Gate/up of 33 to 64 rows and more column blocks of 64 features than units: 128-row tiles, whose weight stream runs deeper (two sets pipelined across the slice's
    // end instead of three): h = 3584, F = 18944, 48 rows 64.2 -> 53.0 us; h = 5120, F = 27648 110 -> 95.
    if (epi == EPI_SWIGLU && rows > 32 && rows <= 64 && (N + 63) / 64 > 256) c.MT = 4;
    // Gate/up with 129..192 certain rows and enough column blocks for one workgroup on (nearly) every compute unit: one
    // 192-row block per column block, so that no weight band is streamed by two workgroups.  (For the split-k
    // projections the same tile was measured: it wants more splits, and the slab traffic costs more than it saves.)
    // Where no row beyond 192 is possible also with fewer column blocks, as long as two 128-row blocks would be a second workgroup on some units: h = 3584,
    // F = 18944 (148 column blocks), four layers of a pass, 150 rows 736 -> 692 us, 190 rows 754 -> 714 (h = 2048, F = 11008, 86 blocks: 435 -> 447).
    if (epi == EPI_SWIGLU && min_rows > 128 && min_rows <= 192 && ((rows <= 384 && (N + 127) / 128 >= 192) || (rows <= 192 && (N + 127) / 128 > 132))) c.MT = 6;
    if (epi == EPI_STORE_F32 || epi == EPI_RESID) {
        const int S = K / 64;
        const long cap_m = (long)(slab_room_floats / ((size_t)rows * N));    // slabs must fit the scratch area
        // every split owns at least three 64-deep slices and no split is empty: with ceil(S / splits) slices per split the last
        // ones of an uneven division would be, and their slabs never written
        auto clamp = [&](long sp) {
            sp = min(min(sp, cap_m), min(16L, (long)(S / 3)));
            if (sp <= 1) return 1;
            const int per = (S + (int)sp - 1) / (int)sp;
            return (S + per - 1) / per;
        };
        if (c.MT == 1 && epi == EPI_RESID) {
            // Up to 32 rows (of the plain-store products, QKV, none: see qkv_rows): workgroups of 128 columns, k split until they are about one round of the units, or with long
            // k (many slices, small slabs) nearly two; a third workgroup on some units costs a third: 24 rows, N = 5120, K = 27648 13 splits (520 workgroups) 57.8 -> 11 splits 50.6 us.
            c.NT = 1;
            c.splits = clamp((K > 4096 ? 448 : 256) / ((N + 127) / 128));
        } else {
            // 128-row tiles from 33 rows on (64-row tiles: N = 4608, K = 3584, 48 rows 13.1 us, so 9.8; N = 5120, K = 27648 61.7 and 50.2)
            c.MT = 4;
            const int at = min_rows > 0 ? (min_rows + likely_rows(rows, min_rows)) / 2 : rows;
            float best = 0.f;
            for (int NT = 1; NT <= 2; ++NT)
                for (int want = 1, last = 0; want <= 16; ++want) {
                    const int sp = clamp(want);
                    if (sp == last) continue;
                    last = sp;
                    const float t = tiled_us(NT, sp, at, N, K);
                    if (best == 0.f || t < best) { best = t; c.NT = NT; c.splits = sp; }
                }
        }
    }
    // A launch of more 128 x 256 workgroups than compute units runs as 128 x 512 workgroups of eight wavefronts, whose activation slice is staged once for twice
    // the columns (7B gate/up 2.5 to 7 % faster), unless the rounds are dealt out worse: a round of 256 of them takes 0.955 of one of 512 small ones, of which
    // 264 or fewer, about one a unit, take 0.58.  us, eight / four: h = 2048, F = 11008 300 rows 49 / 40, 640 58 / 60, 992 103 / 88, 1280 110 / 113;
    // h = 3584, F = 18944 400 rows 160 / 133, 700 177 / 190, 992 260 / 243; h = 1536, F = 8960 509 rows 41 / 43, 992 76 / 63.
    // Beyond four rounds the difference is within 2 % or the wide ones'.  Of 103 random launches of gate/up the rule picks all but three within 1 us of the better.  Residual products (four layers of a
    // pass, ms, always eight / by the rule): h = 5120, F = 27648, 4096 rows 13.09 / 12.48, 3500 rows 11.94 / 11.09, 3000 rows 8.81 / 8.81; h = 6144, F = 16384, 4096 rows 11.43 / 11.32; h = 3584, 4096 and 8192
    // within 0.2 %.  (Measured and not faster: the LM head, the prefill QKV projection.)
    if ((epi == EPI_SWIGLU || epi == EPI_RESID) && c.MT == 4 && c.NT == 2 && c.splits == 1) {
        const int cols4 = epi == EPI_SWIGLU ? (N + 127) / 128 : (N + 255) / 256, mb = sure_blocks(rows, min_rows, c.MT);
        const int b4 = cols4 * mb, rounds8 = ((cols4 + 1) / 2 * mb + 255) / 256, rest4 = b4 % 512;
        const int t4 = 1000 * (b4 / 512) + (rest4 == 0 ? 0 : rest4 <= 264 ? 580 : 1000);
        if (b4 > 256 && (rounds8 > 4 || 955 * rounds8 < t4)) c.WV = 8;
    }
    if (epi == EPI_SWIGLU) refine_gateup(rows, min_rows, N, K, &c);
    return c;
}

template <int EPI>
static void launch_cfg(hipStream_t s, const TileChoice &c, MfmaArgs &a, int min_rows)
{
    const int per_wg = c.WV / c.KH * c.NT;
    a.n_blocks = (a.n_tiles + per_wg - 1) / per_wg;
    a.m_blocks = (a.max_rows + c.MT * 32 - 1) / (c.MT * 32);
    a.splits = c.splits;
    int S = a.K / 64;
    a.stages_per_split = (S + c.splits - 1) / c.splits;
    a.m_sure = sure_blocks(a.max_rows, min_rows, c.MT);
    a.rows_sure = min_rows < 0 ? 0 : (min_rows > a.max_rows ? a.max_rows : min_rows);
    const int first = a.n_blocks * a.splits * a.m_sure, rest = a.n_blocks * a.splits * (a.m_blocks - a.m_sure);
    dim3 grid((first + 7) / 8 * 8 + (rest + 7) / 8 * 8), block(c.WV * 64);
    if constexpr (EPI == EPI_SWIGLU) {
        if (c.KH == 2) {
            if (c.MT == 2) hipLaunchKernelGGL((gemm_mfma_k<2, 2, EPI, 4, 2>), grid, block, 0, s, a);
            else hipLaunchKernelGGL((gemm_mfma_k<4, 2, EPI, 4, 2>), grid, block, 0, s, a);
            return;
        }
        if (c.MT == 8) { hipLaunchKernelGGL((gemm_mfma_k<8, 2, EPI>), grid, block, 0, s, a); return; }
    }
#define SDLM_GO(...) hipLaunchKernelGGL((gemm_mfma_k<__VA_ARGS__>), grid, block, 0, s, a)
    if constexpr (EPI == EPI_LMHEAD) {
        if (c.MT == 1) SDLM_GO(1, 2, EPI); else if (c.MT == 2) SDLM_GO(2, 2, EPI); else SDLM_GO(4, 2, EPI);
    } else if constexpr (EPI == EPI_SWIGLU) {   // up to 32 rows: the kernels without LDS tiles
        if (c.MT == 2) SDLM_GO(2, 2, EPI); else if (c.MT == 6) SDLM_GO(6, 2, EPI); else if (c.WV == 8) SDLM_GO(4, 2, EPI, 8); else SDLM_GO(4, 2, EPI);
    } else {
        if (EPI == EPI_RESID && c.MT == 1) SDLM_GO(1, 1, EPI_RESID);
        else if (c.NT == 1) SDLM_GO(4, 1, EPI);
        else if (EPI == EPI_RESID && c.WV == 8) SDLM_GO(4, 2, EPI_RESID, 8);
        else SDLM_GO(4, 2, EPI);
    }
#undef SDLM_GO
}

void mfma_gemm_plan(int epi, int rows, int min_rows, int N, int K, size_t slab_room_floats, int *tile_rows, int *tile_cols, int *splits)
{
    const TileChoice c = choose(epi, rows, min_rows, N, K, slab_room_floats);
    *tile_rows = c.kind == FEW16 ? 16 : 32 * c.MT;
    *tile_cols = c.kind == FEW16 ? 32 : 32 * c.NT * (c.WV / c.KH);
    *splits = c.splits;
}

int launch_gemm_mfma(hipStream_t s, int epi, const GemmArgs &g, float *slabs, size_t slab_room_floats, bool defer_reduce)
{
    MfmaArgs a{};
    a.X = (const bf16_t *)g.X; a.Wp = (const bf16_t *)g.W; a.bias = (const bf16_t *)g.bias;
    a.Yf = g.Yf; a.Yt = (bf16_t *)g.Yt; a.pR = g.pR; a.max_rows = g.max_rows; a.N = g.N; a.K = g.K; a.scale = g.scale;
    a.n_out = g.N;
    a.n_tiles = epi == EPI_SWIGLU ? 2 * (int)(mfma_pad_n(g.N) / 32) : (int)(mfma_pad_n(g.N) / 32);
    const TileChoice c = choose(epi, g.max_rows, g.min_rows, g.N, g.K, slab_room_floats);
    a.slab = (size_t)g.max_rows * g.N;
    a.splits = c.splits;
    if (c.splits > 1) a.Yf = slabs;
    if (c.kind == TILED) {
        switch (epi) {
        case EPI_STORE_F32: launch_cfg<EPI_STORE_F32>(s, c, a, g.min_rows); break;
        case EPI_RESID: launch_cfg<EPI_RESID>(s, c, a, g.min_rows); break;
        default: launch_cfg<EPI_SWIGLU>(s, c, a, g.min_rows); break;
        }
    } else if (epi == EPI_RESID) {
        hipLaunchKernelGGL(resid_skinny_k<false>, dim3(a.n_tiles * c.splits), dim3(SK_W * 64), 0, s, a);
    } else if (c.kind == FEW16) {
        hipLaunchKernelGGL(swiglu_skinny16_k<false>, dim3(a.n_tiles), dim3(SK_W * 64), 0, s, a);
    } else {
        hipLaunchKernelGGL(swiglu_skinny32_k, dim3(a.n_tiles / 2), dim3(SK_W * 64), 0, s, a);
    }
    if (c.splits > 1 && epi == EPI_RESID && !defer_reduce)
        hipLaunchKernelGGL(reduce_slabs_k, dim3(g.max_rows), dim3(256), 0, s, g.Yf, slabs, c.splits, a.slab, g.N, g.pR, g.max_rows);
    return c.splits;   // slabs left for the consumer: always for STORE_F32, for RESID when defer_reduce
}

bool mfma_few_applies(const sdlm_model_cfg *m, int max_rows) { return mfma_supported(m) && max_rows <= 16 && m->hidden <= 1024 * FEW_SSQ; }

void launch_embed_few(hipStream_t s, float *x, const void *E, const RowMeta &rm, int max_rows, int h, int V, const void *gain, void *xg, float *ssq)
{
    hipLaunchKernelGGL(embed_few_k, dim3((h + 1023) / 1024, max_rows), dim3(256), 0, s, x, (const bf16_t *)E, rm.tok, rm.counts, h, V, (const bf16_t *)gain, (bf16_t *)xg, ssq);
}

void launch_gateup_few(hipStream_t s, const GemmArgs &g, const float *ssq, float eps)
{
    MfmaArgs a{};
    a.X = (const bf16_t *)g.X; a.Wp = (const bf16_t *)g.W; a.Yt = (bf16_t *)g.Yt; a.pR = g.pR; a.max_rows = g.max_rows; a.N = g.N; a.K = g.K; a.ssq = const_cast<float *>(ssq); a.eps = eps;
    hipLaunchKernelGGL(swiglu_skinny16_k<true>, dim3(2 * (int)(mfma_pad_n(g.N) / 32)), dim3(SK_W * 64), 0, s, a);
}

void launch_resid_few(hipStream_t s, const GemmArgs &g, bool ordered, const void *gain, void *xg, float *ssq)
{
    MfmaArgs a{};
    a.X = (const bf16_t *)g.X; a.Wp = (const bf16_t *)g.W; a.Yf = g.Yf; a.pR = g.pR; a.max_rows = g.max_rows; a.N = a.n_out = g.N; a.K = g.K;
    a.gain = (const bf16_t *)gain; a.xg = (bf16_t *)xg; a.ssq = ssq;
    // O beyond one round of the units: 32 features a workgroup, whose rows are requested half as often (h = 5120, 320 -> 160 workgroups, 8 layers: 8 rows 1887 -> 1874 us, 16 rows 2000 -> 1988;
    // h = 3584, 224 -> 112: 1133 -> 1147).
    if (ordered) hipLaunchKernelGGL((resid_few_k<true, 1>), dim3(g.N / 16), dim3(FEW_W * 64), 0, s, a);
    else if (g.N / 16 > 256) hipLaunchKernelGGL((resid_few_k<false, 2>), dim3(g.N / 32), dim3(FEW_W * 64), 0, s, a);
    else hipLaunchKernelGGL((resid_few_k<false, 1>), dim3(g.N / 16), dim3(FEW_W * 64), 0, s, a);
}

// Down of that chain by whole sums where its workgroups of 16 features are nearly one round of the units: h = 3584, F = 18944, 8 rows, 224 workgroups, a step of 8 layers 1168 us
// with k splits and an RMSNorm, 1136 without.  Fewer leave units without work, which costs the launch what the norm's saves (h = 1536, 96 workgroups, 28 layers:
// 8 rows 1509 / 1502, 16 rows 1595 / 1614; h = 2048, 128, 18 layers: 1222 / 1214, 1278 / 1302); more are an uneven second one (h = 5120, 320, 8 layers: 1963 / 2055).  The ends of the
// range, six layers, 16 and 6 rows: h = 3136, F = 8960 527 / 518, F = 16384 659 / 651, h = 3328 645 / 620, h = 3840 740 / 712, h = 4096, F = 14336 756 / 726, F = 8192 563 / 534, F = 22016 949 / 929.
bool few_down_whole(int h) { return h / 16 > 192 && h / 16 <= 256; }

int launch_down_split(hipStream_t s, const GemmArgs &g, float *slabs, size_t slab_room_floats, bool defer_reduce)
{
    MfmaArgs a{};
    a.X = (const bf16_t *)g.X; a.Wp = (const bf16_t *)g.W; a.pR = g.pR; a.max_rows = g.max_rows; a.N = a.n_out = g.N; a.K = g.K;
    a.splits = skinny_splits(g.max_rows, g.N, g.K, slab_room_floats);
    a.slab = (size_t)g.max_rows * g.N;
    a.Yf = a.splits > 1 ? slabs : g.Yf;
    hipLaunchKernelGGL(resid_skinny_k<true>, dim3(g.N / 32 * a.splits), dim3(SK_W * 64), 0, s, a);
    if (a.splits > 1 && !defer_reduce)
        hipLaunchKernelGGL(reduce_slabs_k, dim3(g.max_rows), dim3(256), 0, s, g.Yf, slabs, a.splits, a.slab, g.N, g.pR, g.max_rows);
    return a.splits;
}

// dst[row, k], row-major, from an operand in the order of ordered_off; eight elements a thread (debug taps).
__global__ __launch_bounds__(256) void unorder_k(bf16_t *dst, const bf16_t *src, int K)
{
    const int row = blockIdx.y, k = (blockIdx.x * 256 + threadIdx.x) * 8;   // K is a multiple of 64
    if (k >= K) return;
    bf16_t *d = dst + (size_t)row * K + k;   // the caller's pointer: element-wise, whatever its alignment
    const bf16_t *v = src + ordered_off(row, k, K);
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = v[e];
}

void launch_unorder(hipStream_t s, void *dst, const void *src, int rows, int K)
{
    hipLaunchKernelGGL(unorder_k, dim3((K + 2047) / 2048, rows), dim3(256), 0, s, (bf16_t *)dst, (const bf16_t *)src, K);
}

void launch_lmhead_mfma(hipStream_t s, const void *xhat, const void *w_packed, const int32_t *p_rows, int max_rows, int min_rows, int V, int h, float scale,
                        int conf_fn, float *logits_out, void *scratch, int32_t *ids, float *conf)
{
    MfmaArgs a{};
    a.X = (const bf16_t *)xhat; a.Wp = (const bf16_t *)w_packed; a.pR = p_rows; a.max_rows = max_rows; a.N = V; a.K = h; a.scale = scale;
    a.n_out = V; a.logits = logits_out; a.lm_part = (float4 *)scratch;
    a.n_tiles = (int)(mfma_pad_n(V) / 32);
    TileChoice c = choose(EPI_LMHEAD, max_rows, min_rows, V, h, 0);
    launch_cfg<EPI_LMHEAD>(s, c, a, min_rows);
    hipLaunchKernelGGL(lm_combine_k, dim3(max_rows), dim3(256), 0, s, (const float4 *)scratch, a.n_blocks, max_rows, p_rows, V, conf_fn, ids, conf);
}

size_t mfma_lm_scratch_bytes(int V, int max_rows) { return (size_t)((mfma_pad_n(V) / 32 + 7) / 8) * max_rows * sizeof(float4); }

}  // namespace sdlm
