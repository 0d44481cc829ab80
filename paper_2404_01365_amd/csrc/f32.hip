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
// each, took 89 us where this took 8 for the output of the same prompt; the whole prompt phase of 256 tokens through a
// 1024 x 4096 block 2021 -> 123 us, of 1500 tokens through a bf16 1024 x 4002 block 10046 -> 465 us.)  Operands come out of
// the L2s once per tile, which is what bounds long prompts: they take 64-token tiles as soon as those fill the chip
// (selection from 2048 tokens of a 1024 x 4096 block: 584 us with 32, 472 with 64).
#include "topk_row.h"

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

// Four elements k .. k+3 of a row.  Elements past the end of the contraction are zero on both sides: where rows come an element a load at
// once, else when they are used (fn_cut).  With a select behind every load it was up to the compiler's order whether the loads of the next slices
// were waited for before the MFMAs of these, and 1 to 3 % of a call hung on it; the loop itself reads no slice that is not all there.  Select behind
// the load / so, us: selections of 4000 tokens of 512 x 1400 201 / 172, of 1500 tokens of 2048 x 6000 906 / 820; outputs of 520 tokens of a bf16 4096 x 2004
// block 136 / 130, of 1500 tokens of 2048 x 6000 429 / 430, of 200 tokens of it 84.9 / 87.3.
template <bool BF16, bool VEC>
__device__ __forceinline__ f32x4_f fn_load(const void *row, int k, int K)
{
    f32x4_f v;
    if (VEC) {                // K and the strides are multiples of four, rows aligned for four elements
        const int kc = k < K ? k : 0;       // the load itself is unconditional: a branch around it would make the next one wait
        if (BF16) {
            const uint2 w = *(const uint2 *)((const uint16_t *)row + kc);
            v = (f32x4_f){bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y)};
        } else {
            v = *(const f32x4_f *)((const float *)row + kc);
        }
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

template <bool VEC>
__device__ __forceinline__ f32x4_f fn_cut(f32x4_f v, int k, int K)
{
    if (VEC) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = k < K ? v[e] : 0.0f;
    }
    return v;
}

// ACT: sigma and the row sums of the first contraction; else a plain product.  BBF16: B, the biases and a plain
// product's C are bf16.  MT: 16-token tiles per workgroup.
// WAVES: wavefronts of the workgroup, of which each has every WAVES-th slice.
// CT: its 16-column tiles (two, or one of a plain product).
// SUMS: of a wave's slices, every SUMS-th goes to a sum of its own: eight waves with two add up exactly as sixteen with one.
template <bool ACT, bool GATED, bool BBF16, bool VEC, int MT, int WAVES, int CT = 2, int SUMS = 1>
__device__ __forceinline__ void f32_nt_tile(const F32NtParams &p, int bx, int by, float (*part)[GATED ? 2 : 1][MT * 16][FN_LD])
{
    constexpr int NMAT = GATED ? 2 : 1, ES = BBF16 ? 2 : 4, S = 2;
    static_assert(S % SUMS == 0, "the slices of a step go to the same sums as those of the one before");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, q = lane >> 4;
    const int m0 = bx * (MT * 16), n0 = by * (CT * 16);
    static_assert(CT * 16 == FN_COLS || !ACT, "rowpart has one sum of FN_COLS columns");

    // rows past the end repeat the last one; what they give is not stored
    const float *ar[MT];
    const char *br[NMAT][CT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
        ar[t] = p.A + (int64_t)min(m0 + t * 16 + r16, p.M - 1) * p.lda;
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const int64_t bo = (int64_t)min(n0 + t * 16 + r16, p.N - 1) * p.ldb * ES;
        br[0][t] = (const char *)p.B + bo;
        if (GATED)
            br[NMAT - 1][t] = (const char *)p.Bg + bo;
    }
    f32x4_f acc[SUMS * NMAT][MT][CT];
#pragma unroll
    for (int m = 0; m < SUMS * NMAT; ++m)
#pragma unroll
        for (int t = 0; t < CT * MT; ++t)
            acc[m][t / CT][t % CT] = (f32x4_f){0.0f, 0.0f, 0.0f, 0.0f};

    f32x4_f a0[S][MT], a1[S][MT], b0[S][NMAT][CT], b1[S][NMAT][CT];
// S slices from number s_ on (slices of this wave are WAVES apart)
#define FN_LOAD(a_, b_, s_)                                                                          \
    _Pragma("unroll") for (int u = 0; u < S; ++u)                                                    \
    {                                                                                                \
        const int k_ = (((s_) + u) * WAVES + wave) * FN_K + q * 4;                                \
        _Pragma("unroll") for (int t = 0; t < MT; ++t) a_[u][t] = fn_load<false, VEC>(ar[t], k_, p.K); \
        _Pragma("unroll") for (int t = 0; t < CT * NMAT; ++t)                                        \
            b_[u][t / CT][t % CT] = fn_load<BBF16, VEC>(br[t / CT][t % CT], k_, p.K);                \
    }
#define FN_MFMA(a_, b_)                                                                              \
    _Pragma("unroll") for (int u = 0; u < S; ++u)                                                    \
        _Pragma("unroll") for (int c = 0; c < 4; ++c)                                                \
            _Pragma("unroll") for (int m = 0; m < NMAT; ++m)                                         \
                _Pragma("unroll") for (int t = 0; t < CT * MT; ++t)                                  \
                    acc[u % SUMS * NMAT + m][t / CT][t % CT] =                                       \
                        __builtin_amdgcn_mfma_f32_16x16x4f32(a_[u][t / CT][c], b_[u][m][t % CT][c], acc[u % SUMS * NMAT + m][t / CT][t % CT], 0, 0, 0);

// ... of which some may lie past the end
#define FN_CUT(a_, b_, s_)                                                                           \
    _Pragma("unroll") for (int u = 0; u < S; ++u)                                                    \
    {                                                                                                \
        const int k_ = (((s_) + u) * WAVES + wave) * FN_K + q * 4;                                   \
        _Pragma("unroll") for (int t = 0; t < MT; ++t) a_[u][t] = fn_cut<VEC>(a_[u][t], k_, p.K);    \
        _Pragma("unroll") for (int t = 0; t < CT * NMAT; ++t) b_[u][t / CT][t % CT] = fn_cut<VEC>(b_[u][t / CT][t % CT], k_, p.K); \
    }

    const int steps = ((p.K + FN_K - 1) / FN_K + WAVES - 1) / WAVES;
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
        FN_CUT(a0, b0, s)
        FN_MFMA(a0, b0)
        FN_CUT(a1, b1, s + S)
        FN_MFMA(a1, b1)
    } else {
        FN_CUT(a0, b0, s)
        FN_MFMA(a0, b0)
    }
#undef FN_LOAD
#undef FN_CUT
#undef FN_MFMA

    // lane (column r16, row group q) holds rows 4q .. 4q+3 of every 16 x 16 tile
#pragma unroll
    for (int m = 0; m < SUMS * NMAT; ++m)
#pragma unroll
        for (int t = 0; t < CT * MT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                part[m / NMAT * WAVES + wave][m % NMAT][(t / CT) * 16 + q * 4 + i][(t % CT) * 16 + r16] = acc[m][t / CT][t % CT][i];
    __syncthreads();
    if (!ACT) {               // a thread has one element
        for (int e = tid; e < MT * 16 * CT * 16; e += WAVES * 64) {
            const int row = e / (CT * 16), c = e % (CT * 16), col = n0 + c;
            float t = 0.0f;
#pragma unroll
            for (int w = 0; w < WAVES * SUMS; ++w)
                t += part[w][0][row][c];
            if (m0 + row < p.M && col < p.N)
                store_scalar<BBF16>(p.C, (int64_t)(m0 + row) * p.ldc + col, t + (p.b ? load_scalar<BBF16>(p.b, col) : 0.0f));
        }
        return;
    }
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
                for (int w = 0; w < WAVES; ++w)
                    t += part[w][m][row][c0 + e];
                v[m][e] = t;
            }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int col = n0 + c0 + e;
            if (col < p.N) {
                float u = v[0][e] + (p.b ? load_scalar<BBF16>(p.b, col) : 0.0f);
                if (GATED)
                    u = act_apply(p.act, v[NMAT - 1][e] + (p.bg ? load_scalar<BBF16>(p.bg, col) : 0.0f)) * u;
                else
                    u = act_apply(p.act, u);
                sq = fmaf(u, u, sq);
                if (grow < p.M)
                    store_scalar<BBF16>(p.C, (int64_t)grow * p.ldc + col, u);
            }
        }
        sq = row16_sum(sq);
        if ((tid & 15) == 0 && grow < p.M)
            p.rowpart[(int64_t)grow * p.nt + by] = sq;
    }
}

template <bool ACT, bool GATED, bool BBF16, bool VEC, int MT, int SUMS = 1>
__global__ __launch_bounds__(FN_WAVES * 64) void f32_nt_kernel(F32NtParams p)
{
    __shared__ float part[FN_WAVES * SUMS][GATED ? 2 : 1][MT * 16][FN_LD];
    f32_nt_tile<ACT, GATED, BBF16, VEC, MT, FN_WAVES, 2, SUMS>(p, blockIdx.x, blockIdx.y, part);
}

// Outputs of little work (at most a 32 x 32 tile for every CU): sixteen wavefronts halve the chain of loads, T = 1 has tiles of 16 x 16 (a
// CU takes its two operands in at some 24 B a clock: 64 tokens of 256 x 688 are 16 tiles of 176 KB, or 64 of 88), and the top-k
// of a prompt phase, which needs one CU a sequence and nothing of the product, goes in the first workgroups.  Whole prompt phases, us, eight
// wavefronts and the top-k before / so: 64 tokens of 256 x 688 23.0 / 16.8 (16 x 16 tiles; 21.9 with 32 x 32), 77 of a bf16 512 x 1001 41.7 / 25.6,
// 200 of 1024 x 4096 113 / 103 (832 tiles of 16 x 16, more bytes a CU: 32 x 32).
// Without a top-k to carry (griffin_ff_prompt_out) eight waves may be faster, with two sums each: the bits are those of the prompt phase.  Outputs
// alone, us, eight waves with one sum / with two / sixteen waves: 64 tokens of 64 x 128 4.4 / 5.0 / 4.7 (a slice for each of the eight), 500 of 256 x 688 7.4 / 6.6 /
// 9.9, of 512 x 2048 19.9 / - / 18.6, 250 of 1024 x 4096 36.1 / - / 33.4; of rows that come an element a load, 400 of
// 256 x 255 7.3 / 7.5 / 12.1, of 512 x 697 18.8 / 20.5 / 22.9, of 256 x 801 22.3 / - / 22.6, 77 of 1024 x 4099 91 / 111 / 94.
constexpr int FN_WIDE_WAVES = TOPK_THREADS / 64;
template <bool BBF16, bool VEC, int T, int KPT>
__global__ __launch_bounds__(TOPK_THREADS) void f32_out_topk_kernel(F32NtParams p, TopkJob t)
{
    __shared__ union {
        float part[FN_WIDE_WAVES][1][T * 16][FN_LD];
        TopkShared topk;
    } sh;
    const int b = (int)blockIdx.x - t.rows, mt = (p.M + T * 16 - 1) / (T * 16);
    if (b < 0)
        topk_row<KPT>(sh.topk, t.scores + (int64_t)blockIdx.x * t.n, t.n, t.k, t.idx + (int64_t)blockIdx.x * t.k);
    else
        f32_nt_tile<false, false, BBF16, VEC, T, FN_WIDE_WAVES, T>(p, b % mt, b / mt, sh.part);
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
                   const void *b2, void *Y, int64_t ldy, hipStream_t st, const TopkJob *topk)
{
    F32NtParams p;
    p.A = Z; p.B = W2p; p.Bg = nullptr; p.b = b2; p.bg = nullptr; p.C = Y; p.rowpart = nullptr;
    p.lda = ldz; p.ldb = ldw; p.ldc = ldy;
    p.M = (int32_t)M; p.N = d; p.K = F; p.act = 0; p.nt = f32_ntiles(d);
    const bool tall = f32_tall(M, p.nt);
    const dim3 grid((unsigned)((M + (tall ? 63 : 31)) / (tall ? 64 : 32)), p.nt), block(FN_WAVES * 64);
    const bool vec = F % 4 == 0 && ldz % 4 == 0 && ldw % 4 == 0 && ((uintptr_t)Z & 15) == 0 && ((uintptr_t)W2p & (bf16 ? 7 : 15)) == 0;
    const int64_t tiles = (M + 31) / 32 * p.nt, small = (M + 15) / 16 * ((d + 15) / 16);
    const bool little = tiles <= 256, few = F <= FN_WAVES * FN_K, two_sums = little && !topk && !few && small > 256 && F < (vec ? 1700 : 700);
    if (little && (topk || !few) && !two_sums) {
        const TopkJob t = topk ? *topk : TopkJob{nullptr, nullptr, 0, 0, 0};
#define FN_OUT_GO(BF_, VEC_, KPT_)                                                                                          \
        {                                                                                                                   \
            if (small <= 256) hipLaunchKernelGGL((f32_out_topk_kernel<BF_, VEC_, 1, KPT_>), dim3((unsigned)(t.rows + small)), dim3(TOPK_THREADS), 0, st, p, t); \
            else hipLaunchKernelGGL((f32_out_topk_kernel<BF_, VEC_, 2, KPT_>), dim3((unsigned)(t.rows + tiles)), dim3(TOPK_THREADS), 0, st, p, t); \
        }
#define FN_OUT(KPT_)                                                                                                        \
        {                                                                                                                   \
            if (bf16 && vec) FN_OUT_GO(true, true, KPT_)                                                                    \
            else if (bf16) FN_OUT_GO(true, false, KPT_)                                                                     \
            else if (vec) FN_OUT_GO(false, true, KPT_)                                                                      \
            else FN_OUT_GO(false, false, KPT_)                                                                              \
        }
        TOPK_RIDE(t.n, FN_OUT)
#undef FN_OUT
#undef FN_OUT_GO
        return check_launch("f32_out_topk_kernel");
    }
    if (topk) {
        const int rc = launch_topk(topk->scores, topk->rows, topk->n, topk->k, topk->idx, st);
        if (rc != GRIFFIN_OK)
            return rc;
    }
    if (two_sums) {
#define FN_TWO(BF_, VEC_) hipLaunchKernelGGL((f32_nt_kernel<false, false, BF_, VEC_, 2, 2>), grid, block, 0, st, p);
        if (bf16) { if (vec) FN_TWO(true, true) else FN_TWO(true, false) }
        else      { if (vec) FN_TWO(false, true) else FN_TWO(false, false) }
#undef FN_TWO
        return check_launch("f32_nt_kernel");
    }
    if (bf16) { if (vec) FN_GO(false, false, true, true) else FN_GO(false, false, true, false) }
    else      { if (vec) FN_GO(false, false, false, true) else FN_GO(false, false, false, false) }
#undef FN_GO
    return check_launch("f32_nt_kernel");
}

}  // namespace griffin
