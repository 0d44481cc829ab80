// Prompt phase, first half: the FF activations of every prompt token (Section 3, Eq. 3 applied
// row-wise; Eq. 2 when there is no gate),
//     Z = sigma(X Wg^T + bg) * (X W1^T + b1),
// together with one sum-of-squares partial per (token row, column tile) from which the row
// norms of Section 4.1 are finished elsewhere.
//
// bf16: a dense contraction, so it runs on the matrix cores.  One workgroup (4 wavefronts, 2x2)
// owns a tile of up to 256 tokens x 128 neurons of BOTH products: the X tile is
// staged once in LDS and feeds two sets of v_mfma_f32_16x16x32_bf16 accumulators (gate and up),
// so the epilogue finds g_ij and u_ij in the same lane and applies sigma, the gating product,
// the store of Z and the row sum-of-squares without another pass.  Workgroup ids are remapped so
// that each XCD (ids congruent mod 8 land on the same XCD) walks a contiguous range of tiles and
// reuses W tiles in its own L2.  The main kernel loads tiles straight into LDS; a register-staged
// variant takes the shapes it cannot (d not a multiple of 64).
//
// fp32 blocks: f32.hip.
#include "ff1_kernel.h"

#include <algorithm>
#include <atomic>

namespace griffin {

// compiled in files of their own
template <> int launch_ff1_tiles<GRIFFIN_ACT_SILU>(const Ff1Params &, int, int, bool, bool, int, hipStream_t);
template <> int launch_ff1_tiles<GRIFFIN_ACT_GELU_TANH>(const Ff1Params &, int, int, bool, bool, int, hipStream_t);
template <> int launch_ff1_tiles<GRIFFIN_ACT_RELU>(const Ff1Params &, int, int, bool, bool, int, hipStream_t);
template <> int launch_ff1_two_shapes<GRIFFIN_ACT_SILU>(const Ff1Params &, const Ff1Params &, int, int, hipStream_t);
template <> int launch_ff1_two_shapes<GRIFFIN_ACT_GELU_TANH>(const Ff1Params &, const Ff1Params &, int, int, hipStream_t);
template <> int launch_ff1_two_shapes<GRIFFIN_ACT_RELU>(const Ff1Params &, const Ff1Params &, int, int, hipStream_t);

// Epilogue of the register-staged kernel: sigma, gating, store of Z, row sums of z^2.
// Lane holds column (neuron) l31 of each 32x32 tile and rows (i>>2)*8 + lh*4 + (i&3), i = 0..15.
template <int ACT, bool GATED, int MI>
__device__ __forceinline__ void ff1_mfma_epilogue(const Ff1Params &p, f32x16 (&accU)[MI][2], f32x16 (&accG)[MI][2],
                                                  float (*rs)[64 * MI], int m0, int n0, int tile_n)
{
    constexpr int BM = 64 * MI;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, l31 = lane & 31, lh = lane >> 5;
    float b1j[2], bgj[2];
    int col[2];
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
        col[ni] = n0 + wn * 64 + ni * 32 + l31;
        const int cj = min(col[ni], p.F - 1);
        b1j[ni] = p.b1 ? bf16_bits_to_f32(((const uint16_t *)p.b1)[cj]) : 0.0f;
        bgj[ni] = (GATED && p.bg) ? bf16_bits_to_f32(((const uint16_t *)p.bg)[cj]) : 0.0f;
    }
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int lrow = wm * (32 * MI) + mi * 32 + (i >> 2) * 8 + lh * 4 + (i & 3);
            const int grow = m0 + lrow;
            float sq = 0.0f;
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) {
                const float u = accU[mi][ni][i] + b1j[ni];
                float z;
                if (GATED)
                    z = act_apply_t<ACT>(accG[mi][ni][i] + bgj[ni]) * u;
                else
                    z = act_apply_t<ACT>(u);
                if (col[ni] < p.F) {
                    sq = fmaf(z, z, sq);
                    if (grow < p.M)
                        __builtin_nontemporal_store(z, &p.Z[(int64_t)grow * p.ldz + col[ni]]);
                }
            }
            // sum over the 32 lanes that share this row
            sq = row16_sum(sq);
            sq += __shfl_xor(sq, 16, 64);
            if (l31 == 0)
                rs[wn][lrow] = sq;
        }
    }
    __syncthreads();
    for (int r = tid; r < BM; r += G_THREADS)
        if (m0 + r < p.M)
            p.rowpart[(int64_t)(m0 + r) * p.nt + tile_n] = rs[0][r] + rs[1][r];
}

// ------------------------------------------------------------------------------------ bf16 / MFMA, register-staged
// Fallback for d not a multiple of 64 or row strides too long for 32-bit byte offsets (the k tail is zero-filled in registers, which the
// direct-to-LDS loads cannot do): 16-byte global loads staged through VGPRs into two LDS
// buffers of BK = 64.
template <int ACT, bool GATED, int MI, bool KTAIL>
__global__ __launch_bounds__(G_THREADS) void ff1_bf16_mfma_staged_kernel(Ff1Params p)
{
    constexpr int BM = 64 * MI;
    constexpr int AQ = BM / 32;      // 16-byte chunks of X a thread stages per k-tile
    // [buffer][row][8 chunks of 16 B], chunk c of row r stored at c ^ (r & 7)
    __shared__ u32x4 As[2][BM * 8];
    __shared__ u32x4 B1s[2][G_BN * 8];
    __shared__ u32x4 Bgs[GATED ? 2 : 1][GATED ? G_BN * 8 : 1];
    __shared__ float rs[2][BM];

    // XCD-aware tile order
    const int nblk = p.mt * p.nt;
    const int per_xcd = (nblk + 7) / 8;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= nblk)
        return;
    const int tile_n = logical / p.mt, tile_m = logical % p.mt;
    const int m0 = tile_m * BM, n0 = tile_n * G_BN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // global -> register staging: thread covers chunk `lc` of rows lr + 32 q.  Row offsets are
    // clamped once (rows past the end re-read the last row; their results are never stored).
    const int lr = tid >> 3, lc = tid & 7;
    const uint16_t *xb = (const uint16_t *)p.X + lc * 8;
    const uint16_t *w1b = (const uint16_t *)p.W1 + lc * 8;
    const uint16_t *wgb = GATED ? (const uint16_t *)p.Wg + lc * 8 : nullptr;
    int64_t xo[AQ], wo[4];
#pragma unroll
    for (int q = 0; q < AQ; ++q)
        xo[q] = (int64_t)min(m0 + lr + 32 * q, p.M - 1) * p.ldx;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        wo[q] = (int64_t)min(n0 + lr + 32 * q, p.F - 1) * p.ldw;
    u32x4 ra[AQ], r1[4], rg[4];
    const u32x4 zero4 = {0u, 0u, 0u, 0u};

// global -> registers for the k-tile starting at k0 (with KTAIL, chunks past d read as zero)
#define FF1_LOAD_TILE(k0)                                                     \
    {                                                                         \
        const bool ok_ = !KTAIL || (k0) + lc * 8 < p.d;                       \
        _Pragma("unroll") for (int q = 0; q < AQ; ++q)                        \
            ra[q] = ok_ ? *(const u32x4 *)(xb + xo[q] + (k0)) : zero4;        \
        _Pragma("unroll") for (int q = 0; q < 4; ++q)                         \
        {                                                                     \
            r1[q] = ok_ ? *(const u32x4 *)(w1b + wo[q] + (k0)) : zero4;       \
            if (GATED)                                                        \
                rg[q] = ok_ ? *(const u32x4 *)(wgb + wo[q] + (k0)) : zero4;   \
        }                                                                     \
    }
// registers -> LDS buffer `buf`
#define FF1_STORE_TILE(buf)                                                   \
    {                                                                         \
        _Pragma("unroll") for (int q = 0; q < AQ; ++q)                        \
        {                                                                     \
            const int row_ = lr + 32 * q;                                     \
            As[buf][row_ * 8 + (lc ^ (row_ & 7))] = ra[q];                    \
        }                                                                     \
        _Pragma("unroll") for (int q = 0; q < 4; ++q)                         \
        {                                                                     \
            const int row_ = lr + 32 * q;                                     \
            const int slot_ = row_ * 8 + (lc ^ (row_ & 7));                   \
            B1s[buf][slot_] = r1[q];                                          \
            if (GATED)                                                        \
                Bgs[buf][slot_] = rg[q];                                      \
        }                                                                     \
    }
// LDS -> MFMA operand fragments of k-step kk of buffer `buf`
#define FF1_READ_FRAGS(F_, buf, kk)                                           \
    {                                                                         \
        const int ch_ = (2 * (kk) + lh) ^ sw;                                 \
        _Pragma("unroll") for (int mi = 0; mi < MI; ++mi)                     \
            fa[F_][mi] = As[buf][(wm * (32 * MI) + mi * 32 + l31) * 8 + ch_]; \
        _Pragma("unroll") for (int ni = 0; ni < 2; ++ni)                      \
        {                                                                     \
            f1[F_][ni] = B1s[buf][(wn * 64 + ni * 32 + l31) * 8 + ch_];       \
            if (GATED)                                                        \
                fg[F_][ni] = Bgs[buf][(wn * 64 + ni * 32 + l31) * 8 + ch_];   \
        }                                                                     \
    }
#define FF1_MFMA(F_)                                                          \
    {                                                                         \
        _Pragma("unroll") for (int mi = 0; mi < MI; ++mi)                     \
            _Pragma("unroll") for (int ni = 0; ni < 2; ++ni)                  \
        {                                                                     \
            accU[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(           \
                __builtin_bit_cast(bf16x8, fa[F_][mi]), __builtin_bit_cast(bf16x8, f1[F_][ni]), accU[mi][ni], 0, 0, 0); \
            if (GATED)                                                        \
                accG[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(       \
                    __builtin_bit_cast(bf16x8, fa[F_][mi]), __builtin_bit_cast(bf16x8, fg[F_][ni]), accG[mi][ni], 0, 0, 0); \
        }                                                                     \
    }

    f32x16 accU[MI][2], accG[MI][2];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                accU[mi][ni][i] = 0.0f;
                accG[mi][ni][i] = 0.0f;
            }

    const int KT = (p.d + G_BK - 1) / G_BK;
    const int l31 = lane & 31, lh = lane >> 5, sw = lane & 7;
    u32x4 fa[2][MI], f1[2][2], fg[2][2];      // operand fragments, double-buffered over k-steps

    FF1_LOAD_TILE(0)
    FF1_STORE_TILE(0)
    __syncthreads();
    FF1_READ_FRAGS(0, 0, 0)

    // Per k-tile: the next tile's global loads are issued first; each k-step's MFMAs run on
    // fragments read during the previous k-step; the staged registers go to the other LDS
    // buffer during the last two k-steps; one barrier, then the first fragments of the next
    // tile.
    for (int kt = 0; kt < KT; ++kt) {
        const int buf = kt & 1;
        const bool more = kt + 1 < KT;
        if (more)
            FF1_LOAD_TILE((kt + 1) * G_BK)
        FF1_READ_FRAGS(1, buf, 1)
        FF1_MFMA(0)
        FF1_READ_FRAGS(0, buf, 2)
        FF1_MFMA(1)
        FF1_READ_FRAGS(1, buf, 3)
        FF1_MFMA(0)
        if (more)
            FF1_STORE_TILE(buf ^ 1)
        FF1_MFMA(1)
        __syncthreads();
        if (more)
            FF1_READ_FRAGS(0, buf ^ 1, 0)
    }

#undef FF1_LOAD_TILE
#undef FF1_STORE_TILE
#undef FF1_READ_FRAGS
#undef FF1_MFMA

    ff1_mfma_epilogue<ACT, GATED, MI>(p, accU, accG, rs, m0, n0, tile_n);
}

// ------------------------------------------------------------------------------------ short prompts: d in ranges
// A short prompt has few token tiles, and few neuron tiles times few token tiles leave most of the chip without work
// while the call has to read all the weights (40 tokens of a 4096 x 11008 block: 86 tiles for 256 CUs).  The contraction is
// then cut into ranges of d that each write their raw products (fp32 slabs, [range][up, gate][M][ldu]); this kernel adds
// the ranges in ascending order and applies what the epilogue of the whole product applies: biases, sigma, the gating
// product, Z (and its bf16 copy), the row sums of squares.  A workgroup takes 1024 columns of one token.
struct Ff1ActParams {
    const float *U;
    const void *bg, *b1;
    float *Z, *rowpart;
    uint16_t *Zb;
    int64_t ldu, ldz, ldzb;
    int32_t M, F, act, splits;
};
constexpr int ACT_COLS = 1024;

template <bool GATED>
__global__ __launch_bounds__(256) void ff1_act_kernel(Ff1ActParams p)
{
    __shared__ float part[4];
    const int row = blockIdx.y, j = blockIdx.x * ACT_COLS + threadIdx.x * 4;
    const int64_t slab = (int64_t)p.M * p.ldu;
    float sq = 0.0f;
    if (j < p.F) {
        const float *up = p.U + (int64_t)row * p.ldu + j;
        f32x4_t u = *(const f32x4_t *)up, g = {0.0f, 0.0f, 0.0f, 0.0f};
        if (GATED)
            g = *(const f32x4_t *)(up + slab);
#pragma unroll 4
        for (int s = 1; s < p.splits; ++s) {
            u += *(const f32x4_t *)(up + (int64_t)s * (GATED ? 2 : 1) * slab);
            if (GATED)
                g += *(const f32x4_t *)(up + (int64_t)(2 * s + 1) * slab);
        }
        float z[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int je = min(j + e, p.F - 1);
            const float uu = u[e] + (p.b1 ? bf16_bits_to_f32(((const uint16_t *)p.b1)[je]) : 0.0f);
            if (GATED)
                z[e] = act_apply(p.act, g[e] + (p.bg ? bf16_bits_to_f32(((const uint16_t *)p.bg)[je]) : 0.0f)) * uu;
            else
                z[e] = act_apply(p.act, uu);
            if (j + e < p.F)
                sq = fmaf(z[e], z[e], sq);
        }
        float *zo = p.Z + (int64_t)row * p.ldz + j;
        if (((p.F | (int32_t)p.ldz) & 3) == 0 && ((uintptr_t)p.Z & 15) == 0) {
            *(f32x4_t *)zo = (f32x4_t){z[0], z[1], z[2], z[3]};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (j + e < p.F)
                    zo[e] = z[e];
        }
        if (p.Zb) {                      // only with F, ldzb multiples of 4 (ff1_can_write_zb)
            uint2 h;
            h.x = f32x2_to_bf16x2(z[0], z[1]);
            h.y = f32x2_to_bf16x2(z[2], z[3]);
            *(uint2 *)(p.Zb + (int64_t)row * p.ldzb + j) = h;
        }
    }
    sq = wave_sum(sq);
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0)
        p.rowpart[(int64_t)row * gridDim.x + blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
}

struct Ff1Tile {
    int ti, ni;              // 32 ti tokens x 32 ni neurons
    int64_t tiles;
    double cost;             // of the whole product, in rounds of 256 x 128 tiles on every CU
};

// The shape of the tiles, by what M tokens x n neurons cost on 256 CUs (an Eq. 2 block's tiles are
// twice as wide).  A round of tiles of a shape takes the time FF1_SHAPES states, whatever part of the chip it fills, but for 0.3 of it:
// matrix cores that idle leave the others power to run faster.  Selections (us) with 256 x 128 tiles / the shape this chooses:
// 512 tokens of 4096 x 11008 110 / 100 (256 x 96: 230 tiles instead of 172), 777 of 5120 x 13824 254 / 230 (224 x 128: the last
// tokens need no whole tile), 700 of 4096 x 14336 202 / 169, 1500 of 4096 x 11008 300 / 258, 3000 of 1536 x 6000 160 / 136 (256 x 96),
// 1000 of 1024 x 4096 54 / 46 and 256 of 2048 x 8192 64 / 51 (256 x 64), 40 of 4096 x 11008 72 / 52 (128 x 128 / 64 x 64).
static Ff1Tile ff1_tile(int64_t M, int32_t n, bool gated, bool any_width, bool sums_apart)
{
    const int64_t units = gated ? (n + 31) / 32 : (n + 63) / 64;
    Ff1Tile best = {0, 0, 0, 0.0};
#define FF1_SHAPE_COST(TI_, NI_, COST_)                                                                         \
    if ((gated ? NI_ == 4 || any_width : FF1_SHAPE_EQ2(TI_, NI_)) && (!sums_apart || FF1_SUMS_APART(TI_, NI_))) { \
        const int64_t tiles = ((M + 32 * TI_ - 1) / (32 * TI_)) * ((units + NI_ - 1) / NI_);                    \
        const double cost = COST_ * (0.7 * (double)((tiles + 255) / 256) + 0.3 / 256 * (double)tiles);          \
        if (best.ti == 0 || cost < best.cost)                                                                   \
            best = {TI_, NI_, tiles, cost};                                                                            \
    }
    FF1_SHAPES(FF1_SHAPE_COST)
#undef FF1_SHAPE_COST
    return best;
}

// Two shapes in one launch, of one height: `wide` columns of tiles 128 neurons wide, then `narrow` of 96 (ti = 0: not for this call).  One shape
// seldom fills its last round on 256 CUs; of two, as few wide ones as the rounds of wide tiles alone have room for beside narrow
// ones make the last round a cheaper one, with hardly a CU idle in it.  (A single shape that FF1_SHAPES does not have, 160 tokens or 224 x 96, comes
// out of this too, beyond a round of it: within one the weights' latency counts, 463 tokens of 3072 x 8256 on 195 tiles of 160 x 128 79.2 us, on
// 172 of 256 x 96 76.3.)
// Where the line lies: whole selections and prompt phases, one shape / two (us), by the ratio that the model gives.  0.83 to 0.9: 788 tokens of
// 6144 x 11392 270 / 230, 774 of 4096 x 17088 251 / 218; 0.9 to 0.95: 1026 of 5120 x 13664 302 / 277, 864 of 2048 x 9872 100 / 96; 0.95 to
// 0.97: 1285 of 4096 x 17088 347 / 341, 3748 of 1536 x 7776 207 / 199; 0.97 to 0.98: 491 of 3072 x 18832 138.2 / 137.8, 3979 of 4096 x 17088 935 / 901;
// from 0.99 on as often slower as faster (723 of 2560 x 7392 70.8 / 75.3).  Over 51 random selections and 41 prompt phases that this sends on two shapes
// 0.96 and 0.99 (geometric means; 0.89 to 1.05).  Tiles of 160 tokens are as often slower as faster from 0.933 on already (41 calls, 0.95 to 1.07, mean 1.00; 1404
// tokens of 1536 x 6592 on nine of them 87.3 / 91.5, 419 of 4096 x 10416 0.956).  Going over to the second shape costs a tile's first loads, which nothing
// hides, so short k loops gain nothing: d = 512 31.7 / 31.6 at 0.95, 128 55.2 / 54.7 at 0.94; 768 144 / 142 at 0.97.
constexpr int FF1_TWO_MIN_D = 768;
constexpr double FF1_TWO_LINE = 0.97;
struct Ff1Two {
    int ti;
    int64_t wide, narrow;
    double cost;             // as Ff1Tile's
};
static Ff1Two ff1_two(int64_t M, int32_t n)
{
    Ff1Two best = {0, 0, 0, 0.0};
#define FF1_TWO_COST(TI_, WIDE_, NARROW_)                                                                       \
    {                                                                                                           \
        const int64_t mt = (M + 32 * TI_ - 1) / (32 * TI_), all = (n + 127) / 128;                              \
        const int64_t columns = (all * mt + 255) / 256 * 256 / mt;      /* of tiles, in that many rounds */     \
        int64_t wide = std::min(all, std::max((int64_t)0, (n - 96 * columns + 31) / 32));                       \
        for (int i = 0; i < 2; ++i) {           /* the fewest wide ones, then as many as take no round more */  \
            const int64_t rounds = (wide * mt + 255) / 256, narrow = std::max((int64_t)0, (n - 128 * wide + 95) / 96); \
            const double cost = 0.7 * (WIDE_ * rounds + NARROW_ * std::max((int64_t)0, ((wide + narrow) * mt + 255) / 256 - rounds)) + \
                                0.3 / 256 * (double)mt * (WIDE_ * wide + NARROW_ * narrow);                     \
            if ((best.ti == 0 || cost < best.cost) && (wide * narrow > 0 || (wide + narrow) * mt > 256))        \
                best = {TI_, wide, narrow, cost};                                                               \
            wide = std::min(all, rounds * 256 / mt);                                                            \
        }                                                                                                       \
    }
    FF1_TWO_SHAPES(FF1_TWO_COST)
#undef FF1_TWO_COST
    return best;
}

// The 128-column tiles of an Eq. 2 block, 256 tokens or 128: half the matrix work of a tile of both products, and bound by the L2->L1
// path (~1400 clocks per k-tile against ~2550).
static double ff1_narrow_cost(int64_t M, int32_t n)
{
    const int64_t mt = M > 128 ? (M + 255) / 256 : (M + 127) / 128, tiles = mt * ((n + G_BN - 1) / G_BN);
    return (M > 128 ? 0.55 : 0.42) * (0.7 * (double)((tiles + 255) / 256) + 0.3 / 256 * (double)tiles);
}

// The plain product (128 columns of two matrices, or 256 of one): no more token tiles than of 256 tokens (128, 64 for prompts that
// fit one), each as low as the tokens allow.
struct Ff1Plain { int ti; double cost; };    // cost of a tile, 256 tokens = 1
static Ff1Plain ff1_plain_tile(int64_t M)
{
    const int64_t mt = (M + 255) / 256, need = (M + 32 * mt - 1) / (32 * mt);
    if (M <= 64) return {2, 0.45};
    return need > 7 ? Ff1Plain{8, 1.0} : need > 6 ? Ff1Plain{7, 0.865} : need > 4 ? Ff1Plain{6, 0.785} : Ff1Plain{4, 0.91};
}

template <bool DUAL>
static void launch_plain(const Ff1Params &p, int ti, int grid, hipStream_t st)
{
#define FF1_PLAIN_GO(TI_) hipLaunchKernelGGL((ff1_bf16_mfma_kernel<GRIFFIN_ACT_RELU, true, TI_, 4, true, false, 2, DUAL>), dim3(grid), dim3(G_THREADS), 0, st, p)
    switch (ti) {
    case 2: FF1_PLAIN_GO(2); break;
    case 4: FF1_PLAIN_GO(4); break;
    case 6: FF1_PLAIN_GO(6); break;
    case 7: FF1_PLAIN_GO(7); break;
    default: FF1_PLAIN_GO(8); break;
    }
#undef FF1_PLAIN_GO
}

struct Ff1Plan {
    int splits;              // ranges of d; 1 range: the epilogue of the product does it all
    int per;                 // k-tiles that are summed apart: those of a range, or of one that 128-neuron tiles would have taken
    int room;                // ranges whose slabs the workspace has room for (what 128-neuron tiles would want: queries do not shrink)
    int64_t ldu;             // columns of a slab's row
};

// How many ranges: the cheapest by a cost in microseconds, from (measured) the time of a k-tile on a CU with its item's
// fixed part in k-tiles, the weights at the rate the loop draws them from HBM, the slabs written and read again, and the
// second kernel:
//   * the whole product on 128-neuron tiles: a k-tile 1.15 us (256 tokens; 1.05 with up to 128; an Eq. 2 block's 128-column tiles
//     0.95 / 0.8), 8 (3) k-tiles of prologue and epilogue; on the tiles of ff1_tile see below;
//   * in ranges: the same without sigma in the epilogue (5, 3); up to 64 tokens 1.0 us, 1.25 us where two workgroups share a CU.
// Whole selections of a 4096 x 11008 block, in one range of 256 x 128 (128 x 128) tiles / in 2, 3, 4, 5, 8 ranges (us): 40 tokens 96 / 70, 69, 64, 65, 70;
// 128 tokens 97 / 75, 97, 87, 84, 102; 256 tokens 111 / 88, 120, 114, 112, 138; 512 tokens 115 / 152, 178, ...; of a 2048 x 8192
// block: 40 tokens 58 / 45, 42, 41, 44, 46; 256 tokens 70 / 60, 58, 59, 83, 89; of a 8192 x 8192 Eq. 2 block: 40 tokens
// 127 / 92, 73, 64, 58, 52; 512 tokens 151 / 120, 101, 107, 134, 125.
static Ff1Plan ff1_plan(const griffin_layer &L, int64_t M)
{
    const int KT = L.d / 64;
    Ff1Plan pl = {1, KT, 1, ((int64_t)L.n + 3) & ~(int64_t)3};
    if (L.dtype != GRIFFIN_BF16 || L.d % 64 != 0 || L.ld > (1 << 21) || M < 1 || M > 2048)
        return pl;
    const bool gated = L.Wg != nullptr;
    const int64_t mt = M > 128 ? (M + 255) / 256 : 1;
    const int64_t n128 = mt * ((L.n + G_BN - 1) / G_BN), n256 = mt * ((L.n + 2 * G_BN - 1) / (2 * G_BN));
    const int fix_whole = M > 128 ? 8 : 3, fix_raw = M > 128 ? 5 : 3;
    const double whole_us = M > 128 ? 1.15 : 1.05, whole_narrow_us = M > 128 ? 0.95 : 0.8, kt_us = 1.15 * ff1_plain_tile(M).cost;
    double best = (double)((n128 + 255) / 256) * (KT + fix_whole) * (gated ? whole_us : whole_narrow_us);
    if (!gated)
        best = std::min(best, (double)((n256 + 255) / 256) * (KT + fix_whole) * whole_us);
    const int64_t ntile = gated ? n128 : n256;
    const double hbm_us = (double)(gated ? 2 : 1) * L.n * L.d * 2 / 6.9e6;
    for (int s = 2; s <= 16; ++s) {
        const int per = (KT + s - 1) / s;
        if (per < 4)
            break;
        const int used = (KT + per - 1) / per;
        const double slab = (double)used * (gated ? 2 : 1) * M * pl.ldu * 4;       // bytes
        if (slab > (double)(128 << 20))
            break;
        const int64_t items = ntile * used;
        double t;
        if (M <= 64)
            t = (double)((items + 511) / 512) * (per + fix_raw) * (items > 256 ? 1.25 : 1.0);
        else
            t = (double)((items + 255) / 256) * (per + fix_raw) * kt_us;
        t = (t > hbm_us ? t : hbm_us) + slab * 2 / 7e6 + 5.0;
        if (t < best) {
            best = t;
            pl.splits = pl.room = used;
            pl.per = per;
        }
    }
    // One range on small tiles that keep the ranges' sums apart in registers computes the same, and needs no slabs; a round of them takes
    // 1.25 us a k-tile where few tokens leave it waiting for the weights.  In ranges / so, selections (us): 40 tokens of 4096 x 11008
    // 59.8 / 54.5, 163 of 2048 x 7872 55.2 / 46.6, 32 of 704 x 2384 25.2 / 22.0; but 81 of 7744 x 9040 88.2 / 91.9.  An Eq. 2 block's
    // slabs are half as large, so it has to be cheaper by more: 50 tokens of 1088 x 3072 (compacted, too) 34.3 / 35.1, 34 of 512 x 1328 21.0 / 19.6.
    // So does a single row of tiles of an Eq. 3 block of some shapes, whose rounds wait longer than FF1_SHAPES says when the sums are apart.  In
    // ranges / so: 256 x 64, 196 tokens of 3648 x 9488 73.3 / 80.2, 219 of 3072 x 8816 64.7 / 73.6 (1728 x 3456, 585 tokens 53.2 / 52.3; 220 of 4416 x 15856, 248 tiles, 104.9 / 101.8); 128 x 64, 112
    // of 4096 x 9280 58.1 / 66.9, 111 of 5120 x 13680 82.5 / 87.5 (196 of 3072 x 8176, two rows, 63.9 / 58.8; 108 of 8128 x 12304, five ranges
    // with their slabs, 130.5 / 124.1); 128 x 128 with half of their tokens or less, 47 of 2560 x 17424 68.5 / 73.6, 1 of 3072 x 22800 74.5 / 77.8 (57
    // of 3584 x 19536, two ranges, 91.7 / 86.6); 64 x 64 on a quarter of the chip, 3 of 1536 x 3072 24.1 / 26.9, 4 of 1152 x 3152 23.6 / 24.6 (4 of
    // 1024 x 3360 23.7 / 23.7).
    if (pl.splits > 1) {
        const Ff1Tile t = ff1_tile(M, L.n, gated, true, true);
        double line = gated ? 1.25 : 2.0;
        if (gated && t.ti == 8 && M <= 256 && t.tiles < 224)
            line = 1.8;
        else if (gated && t.ti == 4 && t.ni == 2 && M <= 128 && pl.room <= 3)
            line = 1.45;
        else if (gated && t.ti == 4 && t.ni == 4 && M <= (pl.room == 2 ? 32 : 64))
            line = 1.3;
        else if (gated && t.ti == 2 && t.ni == 2 && t.tiles <= 64)
            line = 1.7;
        if (t.cost * (KT + 8) * line <= best)
            pl.splits = 1;
    }
    return pl;
}

// Does the product go on two shapes of tiles?  (Kernels with biases, and for Eq. 2 blocks, are not compiled; what they would gain is not measured.)
static Ff1Two ff1_takes_two(const griffin_layer &L, int64_t M, const Ff1Plan &pl)
{
    const Ff1Two none = {0, 0, 0, 0.0};
    if (L.dtype != GRIFFIN_BF16 || L.d % 64 != 0 || L.d < FF1_TWO_MIN_D || L.ld > (1 << 21) || !L.Wg || L.b1 || L.bg || M < 1 || pl.room > 1)
        return none;
    const Ff1Two two = ff1_two(M, L.n);
    return two.ti && two.cost < FF1_TWO_LINE * ff1_tile(M, L.n, true, true, false).cost ? two : none;
}

// One range whose tiles are narrower than 128 neurons has more row partials than ff1_ntiles: they go there, too.
size_t ff1_tail_least(const griffin_layer &L, int64_t M)
{
    const Ff1Plan pl = ff1_plan(L, M);
    const size_t slabs = pl.room > 1 ? (size_t)pl.room * (L.Wg ? 2 : 1) * M * pl.ldu * sizeof(float) : 0;
    if (pl.splits > 1)
        return slabs;
    if (L.dtype != GRIFFIN_BF16 || L.d % 64 != 0 || L.ld > (1 << 21) || !L.Wg || M < 1)
        return slabs;
    const int ni = ff1_tile(M, L.n, true, true, pl.room > 1).ni;
    return std::max(slabs, ni < 4 ? (size_t)M * ((L.n + 32 * ni - 1) / (32 * ni)) * sizeof(float) : 0);
}

// ... and so has the product on two shapes
static size_t ff1_two_bytes(const Ff1Two &two, int64_t M) { return (size_t)M * (two.wide + two.narrow) * sizeof(float); }

size_t ff1_tail_bytes(const griffin_layer &L, int64_t M)
{
    const Ff1Two two = ff1_takes_two(L, M, ff1_plan(L, M));
    const size_t least = ff1_tail_least(L, M);
    return two.ti ? std::max(least, ff1_two_bytes(two, M)) : least;
}

int ff1_ntiles(const griffin_layer &L)
{
    return L.dtype == GRIFFIN_BF16 ? (L.n + G_BN - 1) / G_BN : f32_ntiles(L.n);
}

// one workgroup per CU (a multiple of 8, so that every XCD gets the same number), fewer if there are fewer tiles.
// The CU count is asked of the current device at every launch's first use on that device and kept per device.
static int ff1_grid(int nblk, int per_cu = 1)
{
    constexpr int MAX_DEV = 64;
    static std::atomic<int> cus_of[MAX_DEV];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEV)
        dev = -1;
    int cus = dev >= 0 ? cus_of[dev].load(std::memory_order_relaxed) : 0;
    if (cus == 0) {
        int n = 0;
        if (dev < 0 || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8)
            n = 256;
        cus = n & ~7;
        if (dev >= 0)
            cus_of[dev].store(cus, std::memory_order_relaxed);
    }
    const int want = ((nblk + 7) / 8) * 8;
    return want < cus * per_cu ? want : cus * per_cu;
}

// the register-staged kernel takes one tile per workgroup
template <int ACT>
static void launch_staged(Ff1Params p, bool gated, hipStream_t st)
{
    const int bm = p.M > 128 ? 256 : 128;
    p.mt = (p.M + bm - 1) / bm;
    const dim3 grid((p.mt * p.nt + 7) / 8 * 8), block(G_THREADS);
    if (p.M > 128) {
        if (gated) hipLaunchKernelGGL((ff1_bf16_mfma_staged_kernel<ACT, true, 4, true>), grid, block, 0, st, p);
        else hipLaunchKernelGGL((ff1_bf16_mfma_staged_kernel<ACT, false, 4, true>), grid, block, 0, st, p);
    } else {
        if (gated) hipLaunchKernelGGL((ff1_bf16_mfma_staged_kernel<ACT, true, 2, true>), grid, block, 0, st, p);
        else hipLaunchKernelGGL((ff1_bf16_mfma_staged_kernel<ACT, false, 2, true>), grid, block, 0, st, p);
    }
}

// Will the first GEMM's own epilogue leave a bf16 copy of Z beside the fp32 one?  Only the direct-to-LDS
// kernel's usual store path does (bf16 block, d in whole k-tiles, 16-byte aligned rows of Z, biases 8-byte aligned).
bool ff1_can_write_zb(const griffin_layer &L, int64_t ldx, const float *Z, int64_t ldz)
{
    const bool ktail = L.d % 64 != 0 || ldx > (1 << 21) || L.ld > (1 << 21);
    const bool vec = ((L.n | (int32_t)ldz) & 3) == 0 && ((uintptr_t)Z & 15) == 0;
    const bool bias8 = (((uintptr_t)L.b1 | (uintptr_t)L.bg) & 7) == 0;
    return L.dtype == GRIFFIN_BF16 && !ktail && vec && bias8 && ldz <= FF1_LDZ_MAX;
}

// Rows whose stride is a multiple of 8 KB have their k-tile number kt in the same memory channels, all of them.  Where one row of token tiles reads
// the weights at the rate of HBM, each column of tiles therefore begins at another k-tile and goes round.  What counts is the bytes that are
// read, not the stride: rows may be padded or interleaved.  Whole selections with cold weights, all from k-tile 0 / so (us).  Eq. 3: 40 tokens of
// 4096 x 11008 (180 MB) 52 / 46 or 47.6 / 46.2, after where the matrices lie, of 4096 x 14336 64 / 51, 100 of it 81 / 66, 40 of 4096 x 9100 46.5 / 44.1; smaller
// blocks as often lose: 40 of 4096 x 8900 (146 MB) 46.2 / 47.3, 64 of it 49.0 / 46.7, 40 of 8192 x 4400 42.8 / 43.6, of 8192 x 3000 (98 MB) 36.6 / 39.3; nor
// do other strides gain: 40 of 5120 x 13824 60.8 / 62.3.  Rows with room between them gain from 139 MB on (40 and 64 tokens of 4096 x 8500 at a stride of 24 KB 46.2 / 47.2
// and 52.5 / 48.2, 100 of 5120 x 6912 at 16 KB 51.7 / 48.2), below that as often lose as gain (sixteen blocks of 51 to 131 MB, 8 to 250 tokens: 0.96 to 1.02 a block, 0.998 in
// all; 40 of 4096 x 5504, 90 MB, at 24 KB 38.1 / 39.2, 100 of 4096 x 7168, 117 MB, 44.5 / 46.4).
// Eq. 2: 40 and 100 tokens of 8192 x 16384 (268 MB) 84 / 63 and 94 / 74, 200 of 4096 x 20000 (164 MB) 80.6 / 78.7, but 40 of it 55.1 / 56.6.  Ranges of d: 2 tokens of
// 16384 x 2300 (151 MB) 42.8 / 39.3, 100 of 12288 x 3100 51.9 / 50.4.  Outputs (one matrix): 100 tokens of 6144 x 12288 (151 MB) 48.1 / 45.1, 40 of 5120 x 16384 43.8 / 40.7,
// 128 of 7168 x 20480 81 / 75.  With more token tiles the X that an XCD's workgroups share has to come at one time: 260 tokens of
// 4096 x 11008 83.2 / 85.8, 1024 of 5120 x 13824 with a start an XCD 232 / 249.
static int32_t ff1_rotates(const Ff1Params &p, int matrices)
{
    return (p.ldw & 4095) == 0 && p.mt == 1 && (int64_t)p.F * p.d * (2 * matrices) >= (p.ldw == p.d ? 150000000 : 139000000);
}

int launch_ff1(const griffin_layer &L, const void *X, int64_t ldx, int64_t M, float *Z, int64_t ldz,
               float **rowpart, int32_t *nt_out, hipStream_t st, uint16_t *Zb, int64_t ldzb, float *tail, size_t room)
{
    Ff1Params p = {};
    p.X = X; p.Wg = L.Wg; p.W1 = L.W1; p.bg = L.bg; p.b1 = L.b1;
    p.Z = Z; p.rowpart = *rowpart;
    p.Zb = (Zb && ff1_can_write_zb(L, ldx, Z, ldz)) ? Zb : nullptr;
    p.ldzb = ldzb;
    p.ldx = ldx; p.ldw = L.ld; p.ldz = ldz;
    p.M = (int32_t)M; p.F = L.n; p.d = L.d;
    p.splits = 1; p.kt_per_split = p.kt_per_sum = L.d / 64;
    // Z is read again at once by the statistic kernel.  While it fits the 256 MB Infinity Cache, plain stores leave it
    // there for that kernel; a Z several times that size is better sent past the caches (measured, statistic kernel
    // after plain / non-temporal stores: 201 MB of Z 38.3 / 44.6 us, 57 MB 14.5 / 16.4 us, 1.18 GB 284 / 243 us; the
    // product itself takes the same time either way).
    p.z_stream = ((int64_t)M * L.n * 4 > ((int64_t)384 << 20) && ldz <= (1 << 20)) ? 1 : 0;   // (32-bit byte offsets inside a tile)
    p.nt = ff1_ntiles(L);
    const bool gated = L.Wg != nullptr;
    const Ff1Plan pl = ff1_plan(L, M);
    if (tail && pl.splits > 1 && ldx <= (1 << 21)) {
        const int nb = (L.n + ACT_COLS - 1) / ACT_COLS;
        *nt_out = nb;
        int rc;
        if (gated) {
            p.Z = tail; p.ldz = pl.ldu; p.Zb = nullptr; p.z_stream = 0;
            p.splits = pl.splits; p.kt_per_split = pl.per;
            const int ti = ff1_plain_tile(M).ti;
            p.mt = (int32_t)((M + 32 * ti - 1) / (32 * ti));
            p.rotate = ff1_rotates(p, 2);
            launch_plain<true>(p, ti, ff1_grid(p.mt * p.nt * pl.splits, M <= 64 ? 2 : 1), st);
            rc = check_launch("ff1_bf16_mfma_kernel");
        } else {
            rc = launch_gemm_nt_partials(X, ldx, L.W1, L.ld, M, L.n, L.d, pl.splits, pl.per, tail, pl.ldu, st);
        }
        if (rc != GRIFFIN_OK)
            return rc;
        Ff1ActParams a;
        a.U = tail; a.bg = L.bg; a.b1 = L.b1; a.Z = Z; a.rowpart = *rowpart;
        a.Zb = (Zb && ff1_can_write_zb(L, ldx, Z, ldz)) ? Zb : nullptr;
        a.ldu = pl.ldu; a.ldz = ldz; a.ldzb = ldzb;
        a.M = (int32_t)M; a.F = L.n; a.act = L.act; a.splits = pl.splits;
        const dim3 agrid(nb, (unsigned)M);
        if (gated)
            hipLaunchKernelGGL(ff1_act_kernel<true>, agrid, dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL(ff1_act_kernel<false>, agrid, dim3(256), 0, st, a);
        return check_launch("ff1_act_kernel");
    }
    // the direct-to-LDS kernel wants whole 64-element k-tiles and 32-bit byte offsets inside a tile
    const bool staged = L.d % 64 != 0 || ldx > (1 << 21) || L.ld > (1 << 21);
    const Ff1Two two = tail && !staged ? ff1_takes_two(L, M, pl) : Ff1Two{0, 0, 0, 0.0};
    if (two.ti && room >= ff1_two_bytes(two, M)) {
        const int64_t split = std::min((int64_t)L.n, two.wide * 128);
        p.mt = (int32_t)((M + 32 * two.ti - 1) / (32 * two.ti));
        p.rotate = ff1_rotates(p, 2);
        p.rowpart = *rowpart = tail;
        p.nt_row = *nt_out = (int32_t)(two.wide + two.narrow);
        Ff1Params b = p;
        p.F = (int32_t)split; p.nt = (int32_t)two.wide;
        b.F = L.n - p.F; b.nt = (int32_t)two.narrow;
        b.W1 = (const uint16_t *)p.W1 + split * p.ldw; b.Wg = (const uint16_t *)p.Wg + split * p.ldw;
        b.Z = p.Z + split; b.rowpart = p.rowpart + p.nt;
        b.Zb = p.Zb ? p.Zb + split : nullptr;
        const int grid = ff1_grid(p.mt * p.nt_row);
        const int rc = L.act == GRIFFIN_ACT_SILU ? launch_ff1_two_shapes<GRIFFIN_ACT_SILU>(p, b, two.ti, grid, st)
                     : L.act == GRIFFIN_ACT_GELU_TANH ? launch_ff1_two_shapes<GRIFFIN_ACT_GELU_TANH>(p, b, two.ti, grid, st)
                     : launch_ff1_two_shapes<GRIFFIN_ACT_RELU>(p, b, two.ti, grid, st);
        return rc != GRIFFIN_OK ? rc : check_launch("ff1_bf16_two_shapes_kernel");
    }
    Ff1Tile t = {8, 4, 0, 0.0};
    bool wide = false;
    const bool apart = tail && pl.room > 1;
    p.kt_per_sum = apart ? pl.per : L.d / 64;
    if (L.dtype == GRIFFIN_BF16 && !staged && M > 0) {
        if (gated) {
            t = ff1_tile(M, L.n, true, tail != nullptr, apart);
            p.nt = (L.n + 32 * t.ni - 1) / (32 * t.ni);
            if (t.ni < 4)
                p.rowpart = *rowpart = tail;
        } else {
            t = ff1_tile(M, L.n, false, true, apart);
            wide = apart || t.cost < ff1_narrow_cost(M, L.n);
            if (wide)
                p.nt = (L.n + 64 * t.ni - 1) / (64 * t.ni);
            else
                t = {M > 128 ? 8 : 4, 4, 0, 0.0};
        }
        p.mt = (int32_t)((M + 32 * t.ti - 1) / (32 * t.ti));
    }
    p.rotate = ff1_rotates(p, gated ? 2 : 1);
    *nt_out = p.nt_row = p.nt;
    if (M == 0)
        return GRIFFIN_OK;
    if (L.dtype == GRIFFIN_BF16) {
        const int grid = staged ? 0 : ff1_grid(p.mt * p.nt);
        int rc = GRIFFIN_OK;
#define FF1_ACT(ACT_)                                                                          \
    {                                                                                          \
        if (staged) launch_staged<ACT_>(p, gated, st);                                         \
        else rc = launch_ff1_tiles<ACT_>(p, t.ti, t.ni, gated, wide, grid, st);                \
    }
        switch (L.act) {
        case GRIFFIN_ACT_SILU: FF1_ACT(GRIFFIN_ACT_SILU) break;
        case GRIFFIN_ACT_GELU_TANH: FF1_ACT(GRIFFIN_ACT_GELU_TANH) break;
        default: FF1_ACT(GRIFFIN_ACT_RELU) break;
        }
#undef FF1_ACT
        return rc != GRIFFIN_OK ? rc : check_launch("ff1_bf16_mfma_kernel");
    }
    return launch_f32_ff1(L, X, ldx, M, Z, ldz, *rowpart, st);
}

// C[s] = A B^T over the s-th range of the contraction, fp32, for s = 0 .. splits-1, on the
// direct-to-LDS kernel: A [M][K] and B [N][K] bf16 with K a multiple of 64, C [splits][M][ldc], ldc a multiple of 4.
// Used by the prompt-output GEMM (Section 5.1) on a bf16 copy of Z.
bool gemm_nt_partials_ok(int64_t M, int32_t N, int32_t K, int64_t lda, int64_t ldb)
{
    return M >= 1 && M <= (1 << 30) && K % 64 == 0 && N % 4 == 0 && lda % 8 == 0 && ldb % 8 == 0 &&
           lda <= (1 << 21) && ldb <= (1 << 21);
}

// The ranges are priced for tiles of 256 or 128 tokens, one workgroup a CU, whatever launch_plain takes of lower ones: they also decide the workspace
// that a call has to bring, which stays what it was.
void gemm_nt_split_plan(int64_t M, int32_t N, int32_t K, int *splits, int *kt_per_split)
{
    const int bm = M > 128 ? 256 : 128;
    const int64_t ntile = ((M + bm - 1) / bm) * ((N + 2 * G_BN - 1) / (2 * G_BN));
    const int KT = K / 64;
    int best = 1;
    int64_t best_cost = -1;
    for (int s = 1; s <= 16 && s <= KT; ++s) {
        const int per = (KT + s - 1) / s;
        if (s > 1 && per < 16)
            break;
        const int used = (KT + per - 1) / per;
        const int64_t rounds = (ntile * used + 255) / 256;
        // in units of one k-tile on every CU (~1.1 us): 8 k-tiles' worth of prologue and epilogue per item, and
        // every range writes an fp32 slab that the sum reads again (8 bytes per element at ~5 TB/s: 5.4 MB per unit)
        const int64_t slab = (int64_t)used * ((M * N * 8) / 5400000);
        const int64_t cost = rounds * (per + 8) + slab;
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = s;
        }
    }
    const int per = (KT + best - 1) / best;
    *splits = (KT + per - 1) / per;
    *kt_per_split = per;
}

int launch_gemm_nt_partials(const void *A, int64_t lda, const void *B, int64_t ldb, int64_t M, int32_t N, int32_t K,
                            int splits, int kt_per_split, float *C, int64_t ldc, hipStream_t st)
{
    Ff1Params p = {};
    p.X = A; p.Wg = nullptr; p.W1 = B; p.bg = nullptr; p.b1 = nullptr;
    p.Z = C; p.rowpart = nullptr;
    p.Zb = nullptr; p.ldzb = 0;
    p.ldx = lda; p.ldw = ldb; p.ldz = ldc;
    p.M = (int32_t)M; p.F = N; p.d = K;
    p.splits = splits; p.kt_per_split = p.kt_per_sum = kt_per_split;
    p.z_stream = p.nt_row = 0;
    p.nt = (N + 2 * G_BN - 1) / (2 * G_BN);        // 256-column tiles: both sets of accumulators hold columns of B
    const int ti = ff1_plain_tile(M).ti;
    p.mt = (int32_t)((M + 32 * ti - 1) / (32 * ti));
    p.rotate = ff1_rotates(p, 1);
    launch_plain<false>(p, ti, ff1_grid(p.mt * p.nt * splits, M <= 64 ? 2 : 1), st);
    return check_launch("ff1_bf16_mfma_kernel");
}

}  // namespace griffin
