// The contractions that stay in 32 bits: the FF activations of fp32 blocks (Eq. 2 / Eq. 3 row-wise, with the row sums of
// squares of Section 4.1), the prompt's own output of fp32 blocks, and that output of bf16 blocks whose D_ff or strides
// the bf16 tiles cannot take (fp32 Z against bf16 W_2).
//
// C[32 or 64 tokens][32 columns] per workgroup on v_mfma_f32_16x16x4_f32 (fp32 products and sums).  Blocks of this kind are
// small, so what a call costs is the chain of memory latencies: a workgroup of eight wavefronts cuts the contraction into
// slices of 16 elements, wave w takes the slices w, w + 8, ..., straight from global memory into registers, four slices on
// their way at once, and the waves' tiles meet once in LDS.  A lane loads four consecutive elements of its row (16 bytes)
// and component c of them is its operand of the c-th MFMA: the order of the contraction differs from memory order in the
// same way on both sides.  (A 64 x 64 FMA tile staged through LDS in 16-element steps, one latency per step and 11
// workgroups, took 30 us where this takes 7 on 64 tokens of a 256 x 688 block; one thread per output, 688 uncoalesced steps
// each, took 89 us where this takes 8 for the output of the same prompt; the whole prompt phase of 256 tokens through a
// 1024 x 4096 block 2021 -> 123 us, of 1500 tokens through a bf16 1024 x 4002 block 10046 -> 465 us.)  Operands come out of
// the L2s once per tile, which is what bounds long prompts: they take 64-token tiles as soon as those fill the chip
// (selection from 2048 tokens of a 1024 x 4096 block: 584 us with 32, 472 with 64).
#include "common.h"

namespace griffin {

typedef __attribute__((ext_vector_type(4))) float f32x4_f;

constexpr int FN_COLS = 32, FN_WAVES = 8, FN_K = 16, FN_LD = 33;

struct F32NtParams {
    const float *A;          // [M][K] fp32
    const void *B, *Bg;      // [N][K]; Bg: the gate's matrix (Eq. 3)
    const void *b, *bg;      // biases of the columns, or NULL
    void *C;                 // fp32 Z or the output
    float *rowpart;
    int64_t lda, ldb, ldc;
    int32_t M, N, K, act, nt;
};

// four elements k .. k+3 of a row; elements past the end of the contraction are zero on both sides
template <bool BF16, bool VEC>
__device__ __forceinline__ f32x4_f fn_load(const void *row, int k, int K)
{
    f32x4_f v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (VEC) {                // K and the strides are multiples of four, rows aligned for four elements
        const bool in = k < K;
        const int kc = in ? k : 0;          // the load itself is unconditional: a branch around it would make the next one wait
        f32x4_f t;
        if (BF16) {
            const uint2 w = *(const uint2 *)((const uint16_t *)row + kc);
            t = (f32x4_f){bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y)};
        } else {
            t = *(const f32x4_f *)((const float *)row + kc);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = in ? t[e] : 0.0f;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
        {
            const float t = load_scalar<BF16>(row, k + e < K ? k + e : 0);
            v[e] = k + e < K ? t : 0.0f;
        }
    }
    return v;
}

// ACT: sigma and the row sums of the first contraction; else a plain product.  BBF16: B, the biases and a plain
// product's C are bf16.  MT: 16-token tiles per workgroup.
template <bool ACT, bool GATED, bool BBF16, bool VEC, int MT>
__global__ __launch_bounds__(FN_WAVES * 64) void f32_nt_kernel(F32NtParams p)
{
    constexpr int NMAT = GATED ? 2 : 1, ES = BBF16 ? 2 : 4, S = 2;
    __shared__ float part[FN_WAVES][NMAT][MT * 16][FN_LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.x * (MT * 16), n0 = blockIdx.y * FN_COLS;

    // rows past the end repeat the last one; what they give is not stored
    const float *ar[MT];
    const char *br[NMAT][2];
#pragma unroll
    for (int t = 0; t < MT; ++t)
        ar[t] = p.A + (int64_t)min(m0 + t * 16 + r16, p.M - 1) * p.lda;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int64_t bo = (int64_t)min(n0 + t * 16 + r16, p.N - 1) * p.ldb * ES;
        br[0][t] = (const char *)p.B + bo;
        if (GATED)
            br[NMAT - 1][t] = (const char *)p.Bg + bo;
    }
    f32x4_f acc[NMAT][MT][2];
#pragma unroll
    for (int m = 0; m < NMAT; ++m)
#pragma unroll
        for (int t = 0; t < 2 * MT; ++t)
            acc[m][t >> 1][t & 1] = (f32x4_f){0.0f, 0.0f, 0.0f, 0.0f};

    f32x4_f a0[S][MT], a1[S][MT], b0[S][NMAT][2], b1[S][NMAT][2];
// S slices from number s_ on (slices of this wave are FN_WAVES apart)
#define FN_LOAD(a_, b_, s_)                                                                          \
    _Pragma("unroll") for (int u = 0; u < S; ++u)                                                    \
    {                                                                                                \
        const int k_ = (((s_) + u) * FN_WAVES + wave) * FN_K + q * 4;                                \
        _Pragma("unroll") for (int t = 0; t < MT; ++t) a_[u][t] = fn_load<false, VEC>(ar[t], k_, p.K); \
        _Pragma("unroll") for (int t = 0; t < 2 * NMAT; ++t)                                         \
            b_[u][t >> 1][t & 1] = fn_load<BBF16, VEC>(br[t >> 1][t & 1], k_, p.K);                  \
    }
#define FN_MFMA(a_, b_)                                                                              \
    _Pragma("unroll") for (int u = 0; u < S; ++u)                                                    \
        _Pragma("unroll") for (int c = 0; c < 4; ++c)                                                \
            _Pragma("unroll") for (int m = 0; m < NMAT; ++m)                                         \
                _Pragma("unroll") for (int t = 0; t < 2 * MT; ++t)                                      \
                    acc[m][t >> 1][t & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a_[u][t >> 1][c], b_[u][m][t & 1][c], acc[m][t >> 1][t & 1], 0, 0, 0);

    const int steps = ((p.K + FN_K - 1) / FN_K + FN_WAVES - 1) / FN_WAVES;
    FN_LOAD(a0, b0, 0)
    int s = 0;
    for (; s + 2 * S < steps; s += 2 * S) {
        FN_LOAD(a1, b1, s + S)
        FN_MFMA(a0, b0)
        FN_LOAD(a0, b0, s + 2 * S)
        FN_MFMA(a1, b1)
    }
    if (s + S < steps) {
        FN_LOAD(a1, b1, s + S)
        FN_MFMA(a0, b0)
        FN_MFMA(a1, b1)
    } else {
        FN_MFMA(a0, b0)
    }
#undef FN_LOAD
#undef FN_MFMA

    // lane (column r16, row group q) holds rows 4q .. 4q+3 of every 16 x 16 tile
#pragma unroll
    for (int m = 0; m < NMAT; ++m)
#pragma unroll
        for (int t = 0; t < 2 * MT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                part[wave][m][(t >> 1) * 16 + q * 4 + i][(t & 1) * 16 + r16] = acc[m][t >> 1][t & 1][i];
    __syncthreads();
    // thread: two neighbouring columns of one row; the sixteen threads of a row are one DPP row of the wavefront
    const int c0 = (tid & 15) * 2;
#pragma unroll
    for (int half = 0; half < MT / 2; ++half) {
        const int row = half * 32 + (tid >> 4), grow = m0 + row;
        float v[NMAT][2], sq = 0.0f;
#pragma unroll
        for (int m = 0; m < NMAT; ++m)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                float t = 0.0f;
#pragma unroll
                for (int w = 0; w < FN_WAVES; ++w)
                    t += part[w][m][row][c0 + e];
                v[m][e] = t;
            }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int col = n0 + c0 + e;
            if (col < p.N) {
                float u = v[0][e] + (p.b ? load_scalar<BBF16>(p.b, col) : 0.0f);
                if (ACT) {
                    if (GATED)
                        u = act_apply(p.act, v[NMAT - 1][e] + (p.bg ? load_scalar<BBF16>(p.bg, col) : 0.0f)) * u;
                    else
                        u = act_apply(p.act, u);
                    sq = fmaf(u, u, sq);
                }
                if (grow < p.M)
                    store_scalar<BBF16>(p.C, (int64_t)grow * p.ldc + col, u);
            }
        }
        if (ACT) {
            sq = row16_sum(sq);
            if ((tid & 15) == 0 && grow < p.M)
                p.rowpart[(int64_t)grow * p.nt + blockIdx.y] = sq;
        }
    }
}

int f32_ntiles(int32_t n) { return (n + FN_COLS - 1) / FN_COLS; }

// 64-token tiles when there are two for every CU (the gated form's LDS holds one at a time)
static bool f32_tall(int64_t M, int nt) { return (M + 63) / 64 * nt >= 512; }

int launch_f32_ff1(const griffin_layer &L, const void *X, int64_t ldx, int64_t M, float *Z, int64_t ldz, float *rowpart,
                   hipStream_t st)
{
    F32NtParams p;
    p.A = (const float *)X; p.B = L.W1; p.Bg = L.Wg; p.b = L.b1; p.bg = L.bg; p.C = Z; p.rowpart = rowpart;
    p.lda = ldx; p.ldb = L.ld; p.ldc = ldz;
    p.M = (int32_t)M; p.N = L.n; p.K = L.d; p.act = L.act; p.nt = f32_ntiles(L.n);
    const bool tall = f32_tall(M, p.nt);
    const dim3 grid((unsigned)((M + (tall ? 63 : 31)) / (tall ? 64 : 32)), p.nt), block(FN_WAVES * 64);
#define FN_GO(ACT_, GA_, BF_, VEC_)                                                                          \
    {                                                                                                        \
        if (tall) hipLaunchKernelGGL((f32_nt_kernel<ACT_, GA_, BF_, VEC_, 4>), grid, block, 0, st, p);       \
        else hipLaunchKernelGGL((f32_nt_kernel<ACT_, GA_, BF_, VEC_, 2>), grid, block, 0, st, p);            \
    }
    if (L.Wg) FN_GO(true, true, false, true)
    else FN_GO(true, false, false, true)
    return check_launch("f32_nt_kernel");
}

int launch_f32_ff2(const float *Z, int64_t ldz, int64_t M, int32_t F, int32_t d, bool bf16, const void *W2p, int64_t ldw,
                   const void *b2, void *Y, int64_t ldy, hipStream_t st)
{
    F32NtParams p;
    p.A = Z; p.B = W2p; p.Bg = nullptr; p.b = b2; p.bg = nullptr; p.C = Y; p.rowpart = nullptr;
    p.lda = ldz; p.ldb = ldw; p.ldc = ldy;
    p.M = (int32_t)M; p.N = d; p.K = F; p.act = 0; p.nt = f32_ntiles(d);
    const bool tall = f32_tall(M, p.nt);
    const dim3 grid((unsigned)((M + (tall ? 63 : 31)) / (tall ? 64 : 32)), p.nt), block(FN_WAVES * 64);
    const bool vec = F % 4 == 0 && ldz % 4 == 0 && ldw % 4 == 0 && ((uintptr_t)Z & 15) == 0 && ((uintptr_t)W2p & (bf16 ? 7 : 15)) == 0;
    if (bf16) { if (vec) FN_GO(false, false, true, true) else FN_GO(false, false, true, false) }
    else      { if (vec) FN_GO(false, false, false, true) else FN_GO(false, false, false, false) }
#undef FN_GO
    return check_launch("f32_nt_kernel");
}

}  // namespace griffin
