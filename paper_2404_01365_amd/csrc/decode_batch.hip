// Generation phase for a batch of rows: up to 64 rows per pass over the weights (Section 5.3, Eq. 7: one expert set
// for the whole batch; or, with membership words, every row its own set inside one block; Eq. 4-5 through it):
//
//     Z[b][j] = sigma(wg_j . x_b + bg_j) * (w1_j . x_b + b1_j),   Y[b][:] = sum_j Z[b][j] W2[j][:]
//
// With a batch the two lines are skinny dense contractions, so they run on the matrix cores; the weights are
// still read exactly once per pass, so the pass stays bound by HBM.  Two kernels, because the two lines want
// different ownership:
//
//  * ff_batch_gu_kernel: a workgroup takes sixteen neurons at a time.  Its W wavefronts share out the 64-element
//    blocks of a row (wave w has the blocks w, w + W, ...: at any time the workgroup reads one window of W x 128
//    bytes that marches along sixteen rows), and a wave keeps its blocks of all the rows of x in registers, as operand
//    fragments of v_mfma_f32_16x16x32_bf16.  The weights go from global memory straight into registers, whole 128-byte
//    lines of eight neurons an instruction, R blocks ahead (bt_ring); the lanes of two such instructions then trade halves, so that a
//    register holds sixteen neurons as the MFMA wants them: a kilobyte of weights costs one load and one MFMA per sixteen
//    rows of the batch and touches no LDS.  A wave's partial tiles go to LDS; the waves meet as seldom as the LDS allows (a
//    barrier per group would tie their load streams to the slowest: 75 us a masked call instead of 71 on 4096 x 14336), add the
//    tiles in wave order, apply sigma, the gating product and the membership bits, and store Z.  Workgroups start at different
//    blocks, so that row strides of a power of two do not send them all to the same memory channels at a time.
//    Measured on the gate and up rows (medians of the kernel trace, each with the ~4 us of a dependent dispatch in it): 5120 x 6912 (142 MB),
//    16 rows 27.8 us, 3072 x 12288, 40 rows 32, 4096 x 14336 masked 40 to 41; 30.6, 34.6 and 42.8 before x came along with the first group
//    and the loads past the last one were cut to a line.  Before that, and each against the form then: 16 rows of 5120 x 6912 31 (34 with five blocks
//    ahead; 38 when rows were streamed through LDS two neurons at a time with two of sixteen MFMA columns in use; 42 with loads of sixteen
//    half lines instead of eight whole ones).
//  * ff_batch_down_kernel: the second line.  Giving every workgroup all d columns would cost one [rows][d] partial per
//    workgroup, so the work is cut in two directions: a workgroup owns 512 columns and one of NR ranges of neurons, and
//    writes one [rows][512] partial into the partial-row buffer that the single-row path uses (NR rows per batch row).
//
// Z is kept in the layout in which the second kernel's MFMAs want it.  Five rows and more at widths of whole 1 KB pieces up to 5120: bf16
// hi + lo pairs (their sum has fp32's accuracy to 2^-17; both are fed), [n/8][tile of 16 rows][hi, lo][16 rows][8 neurons].  At all
// other widths, and for fewer rows, Z stays in fp32, as it is in decode.hip: [n/8][tile][two halves][16 rows][4 neurons].
// The partial rows are added in a fixed order by ff_decode_reduce_kernel (decode.hip).
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace griffin {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_b;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_b;
typedef __attribute__((ext_vector_type(4))) float f32x4_b;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_b;
typedef __attribute__((address_space(3))) void lds_void_b;
typedef __attribute__((address_space(1))) const void gbl_cvoid_b;

constexpr int BT_ROWS = 16;              // rows of x per MFMA tile
constexpr int BT_MAX_T = 4;              // tiles per pass
constexpr int BT_MAX_N = 32768;          // neurons: a pass keeps the Z of all of them, and a partial row per range of a few hundred,
                                         // which for wider blocks is far more than rows taken four at a time need (64 rows of
                                         // 4096 x 65536: 147 MB against 32)
constexpr int BT_WAVES = 8;              // waves per workgroup of the first kernel at the most
constexpr int BT_COLS = 512;             // columns per workgroup of the second kernel
constexpr int BT_WAVES2 = 8;             // waves per workgroup of the second kernel (64 columns each)

struct BatchParams {
    const void *Wg, *W1, *W2, *bg, *b1;
    const void *x;           // [rows][d] bf16
    void *z;                 // fragments of Z (see above)
    float *part;             // [rows][NR][d] fp32
    int64_t ld;
    int32_t d, n, act, rows; // rows <= 16 T
    int32_t exact;           // Z stays in fp32
    int32_t W, P, NB;        // waves per workgroup and workgroups of the first kernel, groups between two meetings of the waves
    int32_t NR, CS;          // neuron ranges x column slices of the second kernel
    const uint32_t *mask;    // [tile][n], bit b set if row b of the tile uses the neuron; NULL: every row uses all
};

// cache policy of the weight stream: read once, so non-temporal (135 MB in a bare read loop: 20.4 us against 23-24 us)
constexpr int BT_NT = 2;

constexpr int bt_vmcnt(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// Blocks of a wave that are on their way at once, a divisor of S (the ring's registers have to be named at compile time).  Two blocks of an
// Eq. 3 block are 64 KB per CU; four or five, 128 to 160 KB, are slower: whole calls of sixteen rows of 5120 x 6912 54.4 / 52.1 us with two, of
// 7680 x 7000 76.5 / 74.8, eight of 4096 x 5504 37.9 / 36.8, the masked pass of 4096 x 14336 70.4 / 69.6.
constexpr int bt_ring(bool gated, int S, int T)
{
    if (gated || T > 1)
        return 2;
    return S % 4 == 0 ? 4 : S % 3 == 0 ? 3 : S % 5 == 0 ? 5 : 2;
}

template <bool GATED, int S, int T>
__global__ __launch_bounds__(BT_WAVES * 64) void ff_batch_gu_kernel(BatchParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char bt_smem[];      // [NB][W][T][NMAT] tiles of 1 KB
    constexpr int NMAT = GATED ? 2 : 1, R = bt_ring(GATED, S, T);
    static_assert(S % R == 0, "the ring of a group must end where it began");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const int W = p.W, rot = (int)(blockIdx.x >> 3) % S;

    // Groups of this workgroup: sixteen neurons at a time round-robin over the chip while every workgroup still gets
    // sixteen; what is left is dealt out in pairs, so that no workgroup has more than two neurons more than another.
    // (The pairs cover the neurons rounded up to eight: the second kernel reads zeros there.)
    const int pairs = ((p.n + 7) >> 3) * 4;
    const int full = pairs / (8 * p.P), rest = pairs - full * 8 * p.P;
    const int r_lo = (int)((int64_t)rest * blockIdx.x / p.P), r_hi = (int)((int64_t)rest * (blockIdx.x + 1) / p.P);
    const int ngroups = full + (r_hi > r_lo ? 1 : 0);
    if (ngroups == 0)
        return;
#define BT_FIRST(g_) ((g_) < full ? ((g_) * p.P + (int)blockIdx.x) * 16 : full * p.P * 16 + r_lo * 2)
#define BT_COUNT(g_) ((g_) < full ? 16 : 2 * (r_hi - r_lo))

    // Block s of this wave: elements BT_K0(s) .. + 63 of a row, of which those from (s W + wave) * 64 on count: a last block that
    // d cuts off, or that is not there, is moved back to the end of the row, and what another block has already is zero
    // on both sides.  (All of it scalar.)
#define BT_BLK(s_) ((((s_) + rot < S ? (s_) + rot : (s_) + rot - S) * W + wave) * 64)
#define BT_K0(s_) min(BT_BLK(s_), p.d - 64)
#define BT_IN(s_, h_) (BT_K0(s_) + (q + 4 * (h_)) * 8 >= BT_BLK(s_))
    const bool tail = S * W * 64 > p.d;

    // lanes of neurons that are not there repeat the last one of the group
    u32x4_b wb[R][NMAT][2];
#define BT_ROW(g_, h_) ((int64_t)min(BT_FIRST(g_) + min((r16 & 7) + 8 * (h_), BT_COUNT(g_) - 1), p.n - 1) * p.ld + (q + 4 * (r16 >> 3)) * 8)
#define BT_LOAD(u_, s_, row_)                                                                        \
    {                                                                                                \
        _Pragma("unroll") for (int h = 0; h < 2; ++h)                                                \
        {                                                                                            \
            const int k_ = BT_K0(s_);                                                                \
            wb[u_][0][h] = __builtin_nontemporal_load((const u32x4_b *)((const uint16_t *)p.W1 + row_[h] + k_)); \
            if (GATED)                                                                               \
                wb[u_][NMAT - 1][h] = __builtin_nontemporal_load((const u32x4_b *)((const uint16_t *)p.Wg + row_[h] + k_)); \
        }                                                                                            \
    }
// bare: the loads of the next blocks stay in flight
#define BT_BARRIER()                                                                                 \
    {                                                                                                \
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                                           \
        __builtin_amdgcn_s_barrier();                                                                \
        asm volatile("" ::: "memory");                                                               \
    }
    int64_t row[2] = {BT_ROW(0, 0), BT_ROW(0, 1)};

    // x: fragment (tile t, block s, half h): row t * 16 + r16, elements (q + 4 h) * 8 .. + 7 of the block.  Rows beyond the batch
    // repeat the last one; their Z is set to zero where it is stored.  Whole lines of eight rows a load, and halves that change places, as
    // the weights do it.  The fragments of a block come with its weights of the first group: with all of x in front (295 KB a CU for 40 rows of
    // 3072) the first MFMA came 6.3 us into the kernel, 4.2 with 16 rows of 4096; so it comes after 2.8 and 2.3.
    u32x4_b xa[T][S][2];
    // byte offsets of this lane's rows: of the first eight of a tile, and of the last tile's, where rows may be missing
    const uint32_t xo = (uint32_t)((r16 & 7) * p.d + (q + 4 * (r16 >> 3)) * 8) * 2;
    uint32_t xl[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
        xl[h] = (uint32_t)(min((T - 1) * BT_ROWS + (r16 & 7) + 8 * h, p.rows - 1) * p.d + (q + 4 * (r16 >> 3)) * 8) * 2;
#define BT_LOAD_X(s_)                                                                                \
    _Pragma("unroll") for (int t = 0; t < T; ++t)                                                    \
        _Pragma("unroll") for (int h = 0; h < 2; ++h)                                                \
        {                                                                                            \
            const char *b_ = (const char *)p.x + (int64_t)((t < T - 1 ? (t * BT_ROWS + 8 * h) * p.d : 0) + BT_K0(s_)) * 2; \
            xa[t][s_][h] = *(const u32x4_b *)(b_ + (t < T - 1 ? xo : xl[h]));                        \
        }
// the halves of two loads change places: then a register holds sixteen rows (a DPP row holds eight of each)
#define BT_SWAP(lo_, hi_)                                                                            \
    _Pragma("unroll") for (int e = 0; e < 4; ++e)                                                    \
    {                                                                                                \
        const int a_ = (int)lo_[e], b_ = (int)hi_[e];                                                \
        lo_[e] = (uint32_t)__builtin_amdgcn_update_dpp(a_, b_, 0x128, 0xF, 0xC, false);   /* lanes 8-15: b of lanes 0-7 */ \
        hi_[e] = (uint32_t)__builtin_amdgcn_update_dpp(b_, a_, 0x128, 0xF, 0x3, false);   /* lanes 0-7: a of lanes 8-15 */ \
    }
#pragma unroll
    for (int s = 0; s < R; ++s) {
        BT_LOAD(s, s, row)
        BT_LOAD_X(s)
    }
    f32x4_b acc[T][NMAT];
    // the blocks of one group; behind the last block the loads of the next group's first ones are on their way
    auto stream = [&](auto first, const int g) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int m = 0; m < NMAT; ++m)
                acc[t][m] = (f32x4_b){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S; ++s) {
#pragma unroll
            for (int m = 0; m < NMAT; ++m)
                BT_SWAP(wb[s % R][m][0], wb[s % R][m][1])
            if (first) {
#pragma unroll
                for (int t = 0; t < T; ++t)
                    BT_SWAP(xa[t][s][0], xa[t][s][1])
            }
            if (tail) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bool in = BT_IN(s, h);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
#pragma unroll
                        for (int m = 0; m < NMAT; ++m)
                            wb[s % R][m][h][e] = in ? wb[s % R][m][h][e] : 0u;
                        if (first) {
#pragma unroll
                            for (int t = 0; t < T; ++t)
                                xa[t][s][h][e] = in ? xa[t][s][h][e] : 0u;
                        }
                    }
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int m = 0; m < NMAT; ++m)
#pragma unroll
                    for (int t = 0; t < T; ++t)
                        acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_b, wb[s % R][m][h]),
                                                                            __builtin_bit_cast(bf16x8_b, xa[t][s][h]), acc[t][m], 0, 0, 0);
            if (s + R < S) {
                BT_LOAD(s % R, s + R, row)
                if (first)
                    BT_LOAD_X(s + R)
            } else {
                // past the last group every lane loads the same few bytes: its own blocks once more were a tenth of all that was read
                if (s + R == S) {
                    row[0] = g + 1 == ngroups ? 0 : BT_ROW(g + 1, 0);
                    row[1] = g + 1 == ngroups ? 0 : BT_ROW(g + 1, 1);
                }
                BT_LOAD(s % R, s + R - S, row)
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    stream(std::true_type{}, 0);
    for (int g = 0;;) {
        // the waves' tiles of the group: lane holds row (of the batch) r16 and neurons 4q .. 4q+3
        const int gi = g % p.NB;
        unsigned char *buf = bt_smem + gi * (W * T * NMAT * 1024) + lane * 16;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int m = 0; m < NMAT; ++m)
                *(f32x4_b *)(buf + ((wave * T + t) * NMAT + m) * 1024) = acc[t][m];
        if (gi == p.NB - 1 || g == ngroups - 1) {
            // the waves meet: the tiles of the last NB groups are shared out over them
            BT_BARRIER()
            for (int i = wave; i < (gi + 1) * T; i += W) {
                const int ge = g - gi + i / T, t = i % T;
                buf = bt_smem + (i / T) * (W * T * NMAT * 1024) + lane * 16;
                f32x4_b u = {0.f, 0.f, 0.f, 0.f}, gt = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
                for (int w = 0; w < W; ++w) {
                    u += *(const f32x4_b *)(buf + ((w * T + t) * NMAT) * 1024);
                    if (GATED)
                        gt += *(const f32x4_b *)(buf + ((w * T + t) * NMAT + NMAT - 1) * 1024);
                }
                const int j0 = BT_FIRST(ge) + q * 4;
                const int cnt = BT_COUNT(ge) - q * 4;           // neurons of this lane, an even number
                if (cnt > 0) {
                    float zv[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int j = min(j0 + i, p.n - 1);
                        float uu = u[i];
                        if (p.b1) uu += bf16_bits_to_f32(((const uint16_t *)p.b1)[j]);
                        float z;
                        if (GATED) {
                            float gg = gt[i];
                            if (p.bg) gg += bf16_bits_to_f32(((const uint16_t *)p.bg)[j]);
                            z = act_apply(p.act, gg) * uu;
                        } else {
                            z = act_apply(p.act, uu);
                        }
                        // beyond the block or the batch, or not in this row's own expert set: no part in the sum (-0, which no other z is)
                        const bool out = j0 + i >= p.n || t * BT_ROWS + r16 >= p.rows || (p.mask && !((p.mask[(int64_t)t * p.n + j] >> r16) & 1u));
                        zv[i] = out ? -0.0f : z + 0.0f;
                    }
#pragma unroll
                    for (int i = 0; i < 4; i += 2)
                        if (i < cnt) {
                            const int j = j0 + i;
                            char *zo = (char *)p.z + ((int64_t)(j >> 3) * T + t) * 512;
                            if (p.exact) {
                                *(float2 *)(zo + ((j >> 2) & 1) * 256 + r16 * 16 + (j & 3) * 4) = make_float2(zv[i], zv[i + 1]);
                            } else {
                                const uint32_t hi = f32x2_to_bf16x2(zv[i], zv[i + 1]);
                                *(uint32_t *)(zo + r16 * 16 + (j & 7) * 2) = hi;
                                *(uint32_t *)(zo + 256 + r16 * 16 + (j & 7) * 2) = f32x2_to_bf16x2(zv[i] - bf16_lo(hi), zv[i + 1] - bf16_hi(hi));
                            }
                        }
                }
            }
        }
        if (++g == ngroups)
            break;
        if (gi == p.NB - 1)
            BT_BARRIER()                 // the tiles may be written again
        stream(std::false_type{}, g);
    }
#undef BT_BARRIER
#undef BT_SWAP
#undef BT_LOAD_X
#undef BT_BLK
#undef BT_K0
#undef BT_IN
#undef BT_FIRST
#undef BT_COUNT
#undef BT_ROW
#undef BT_LOAD
}

// Y partials on the matrix cores: workgroup (nr, cs) owns neurons [j_lo, j_hi) (bounds on
// multiples of 8) and columns cs*512 .. +511; wave w owns 64 of the columns (four 16-column MFMA tiles).
//   D[16 rows of the batch][16 columns] += A[16][32 neurons] * B[32 neurons][16 columns]
// A is Z: the workgroup's range of the fragments that the first kernel left is copied into LDS.
// B is W2, whose memory order (columns
// contiguous) is the transpose of what an MFMA operand wants (neurons contiguous per lane):
// every wave brings its own 32-neuron x 64-column pieces (whole 128-byte lines, 8 rows per
// LDS-DMA instruction) into a private LDS ring and gathers the operands with 16-bit LDS reads, once for all tiles of rows.
// No wave waits for another after the first barrier.
// Ring slots per wave: the pieces of one step are on their way while those of another are used, 32 KB a CU.  With three (64 KB) whole
// calls of 16 rows of 1024 x 5504 take 19.5 us (18.7 with two), 40 of 3072 x 12288 63.3 (61.9), 60 of 2048 x 9000 48.9 (47.3), 16 of 5120 x 6912
// 52.2 (51.5); the masked pass of 4096 x 14336 is the same either way.  With Z in fp32: 50 of 2176 x 10610 90.2 (88.3), of its Eq. 2 block 77.1
// (75.0), 30 of 1280 x 6425 31.3 (30.2), 11 of 6144 x 6734 57.5 (56.9), 16 of 7680 x 7000 75.9 (75.0).
constexpr int BD_DEPTH = 2;
constexpr int BD_REGION = 66;            // 16-byte units per 8-row region: 1 KB of rows + 32 B, so that the four
                                         // regions a gather touches (rows 8q + i) start on different LDS banks
constexpr int BD_SLOT = 4 * BD_REGION;   // a slot: 32 rows x 128 B in four regions
constexpr int BD_RING = BT_WAVES2 * BD_DEPTH * BD_SLOT * 16;    // bytes: 66 KB
// neurons of a range before rounding to multiples of 8: its fragments, 64 T bytes a neuron in steps of 32, go into the
// LDS beside the ring, 61 KB of it (480 with one tile, 472, 312 and 216 with two, three and four)
constexpr int BD_Z_BYTES = 62464;
constexpr int bd_range(int T) { return T == 1 ? 480 : BD_Z_BYTES / (64 * T) / 32 * 32 - 8; }
static_assert(bd_range(1) + 8 + 31 <= BD_Z_BYTES / 64 && BD_Z_BYTES + BD_RING <= 160 * 1024, "the range's fragments fit beside the ring");

//
// EXACT: Z is fp32, split into the three bf16 that hold its 24 bits.  (v_mfma_f32_16x16x4_f32 takes Z as it is, for five times the
// matrix time: whole calls of 50 rows of 2176 x 10610 106 us against 93, 30 rows of 1280 x 6425 33.0 against 29.2, 11 rows of
// 6144 x 6734 63.0 against 58.2; with pairs, 17 bits, they take 85, 27.2 and 56.7.)  A weight that is not finite counts only for the rows that use its
// neuron, as it does when every row reads its own neurons: a step that holds one (no step of a sound model does) takes
// these weights out of the MFMAs, leaving a finite one of their sign, and adds their products lane by lane.
template <int T, bool EXACT>
__global__ __launch_bounds__(BT_WAVES2 * 64) void ff_batch_down_kernel(BatchParams p)
{
    constexpr uint32_t NO_Z = EXACT ? 0x80000000u : 0u;
    extern __shared__ __attribute__((aligned(16))) unsigned char bt_smem[];     // the ring, then the fragments of Z
    u32x4_b *const ring_s = (u32x4_b *)bt_smem;
    const uint32_t zs_a = (uint32_t)(uintptr_t)(lds_void_b *)(bt_smem + BD_RING);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nr = blockIdx.x / p.CS, cs = blockIdx.x % p.CS;
    const int j_lo = (int)((int64_t)p.n * nr / p.NR) & ~7;
    const int j_hi = nr == p.NR - 1 ? p.n : ((int)((int64_t)p.n * (nr + 1) / p.NR) & ~7);
    const int range = j_hi - j_lo;                 // <= bd_range(T) + 8 by the choice of NR
    const int S = (range + 31) >> 5;

    const int bq = lane & 15, q = lane >> 4;
    const int c0 = cs * BT_COLS + wave * 64;
    u32x4_b *ring = ring_s + wave * (BD_DEPTH * BD_SLOT);
    const uint32_t ring_a = (uint32_t)(uintptr_t)(lds_void_b *)ring;
    const uint32_t za = zs_a + (uint32_t)(q * (T * 512) + bq * 16);
    const uint16_t *w2 = (const uint16_t *)p.W2 + min(c0 + (lane & 7) * 8, p.d - 8);    // columns past d repeat the last eight
    const int lrow = lane >> 3;
// the four LDS-DMA instructions of step s_: rows 8u .. 8u+7 of its 32 neurons, 128 bytes per row (past the last step all take
// row 0: the last step's once more, a step of the ten that 40 rows of 3072 x 12288 have, is read for nothing)
#define BD_ISSUE(s_)                                                                                         \
    _Pragma("unroll") for (int u = 0; u < 4; ++u)                                                            \
    {                                                                                                        \
        const int row_ = (s_) < S ? min(j_lo + (s_) * 32 + u * 8 + lrow, p.n - 1) : 0;                       \
        __builtin_amdgcn_global_load_lds((gbl_cvoid_b *)(w2 + (int64_t)row_ * p.ld),                         \
                                         (lds_void_b *)(ring + ((s_) % BD_DEPTH) * BD_SLOT + u * BD_REGION), 16, 0, BT_NT); \
    }
    f32x4_b acc[T][4];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            acc[t][c] = (f32x4_b){0.f, 0.f, 0.f, 0.f};
    // LDS accesses by inline asm here and below: those the compiler knows about would wait for every LDS-DMA in flight.
    // The range's fragments (32 T units of 16 bytes per eight neurons, zero beyond the range) go straight into the LDS, all of them at
    // once, and the first pieces of W2 leave right behind them.  (Through registers, four loads a thread at a time, the prologue took 2.5 us
    // with one tile and 3.8 with three.)
    const u32x4_b *zg = (const u32x4_b *)p.z + (int64_t)(j_lo >> 3) * (32 * T);
    const int units = ((range + 7) >> 3) * (32 * T), units_all = S * 4 * (32 * T);
    for (int u0 = wave * 64; u0 < units; u0 += BT_WAVES2 * 64)
        if (u0 + lane < units)
            __builtin_amdgcn_global_load_lds((gbl_cvoid_b *)(zg + u0 + lane), (lds_void_b *)(bt_smem + BD_RING + u0 * 16), 16, 0, 0);
#pragma unroll
    for (int s = 0; s < BD_DEPTH - 1; ++s)
        BD_ISSUE(s)
    for (int u = units + tid; u < units_all; u += BT_WAVES2 * 64)
        asm volatile("ds_write_b128 %0, %1" :: "v"(zs_a + (uint32_t)(u * 16)), "v"((u32x4_b){NO_Z, NO_Z, NO_Z, NO_Z}) : "memory");
    __builtin_amdgcn_s_waitcnt(bt_vmcnt((BD_DEPTH - 1) * 4));       // the fragments have landed
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (S > 0) {                 // an empty range (very few neurons) still writes its zero partial
    const uint32_t gat = (uint32_t)(q * BD_REGION * 16 + bq * 2);   // row 8q of the slot (region q), column bq of tile 0
    for (int s = 0; s < S; ++s) {
        BD_ISSUE(s + BD_DEPTH - 1)
        __builtin_amdgcn_s_waitcnt(bt_vmcnt((BD_DEPTH - 1) * 4));   // the pieces of step s have landed
        const uint32_t slot = ring_a + (uint32_t)((s % BD_DEPTH) * BD_SLOT * 16) + gat;
        u32x4_b ah[T], al[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            asm volatile("ds_read_b128 %0, %1" : "=v"(ah[t]) : "v"(za + (uint32_t)(s * (T * 2048) + t * 512)));
            asm volatile("ds_read_b128 %0, %1" : "=v"(al[t]) : "v"(za + (uint32_t)(s * (T * 2048) + t * 512 + 256)));
        }
        // eight 16-bit reads per 16-column tile into eight registers (two reads in flight into the
        // halves of one register do not merge), packed in pairs afterwards; all four tiles' reads are
        // issued before the one wait
        uint32_t e[4][8];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                asm volatile("ds_read_u16 %0, %1" : "=v"(e[c][i]) : "v"(slot + (uint32_t)(c * 32 + i * 128)));
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(ah[0]), "+v"(al[0]),
                     "+v"(e[0][0]), "+v"(e[0][1]), "+v"(e[0][2]), "+v"(e[0][3]), "+v"(e[0][4]), "+v"(e[0][5]), "+v"(e[0][6]), "+v"(e[0][7]),
                     "+v"(e[1][0]), "+v"(e[1][1]), "+v"(e[1][2]), "+v"(e[1][3]), "+v"(e[1][4]), "+v"(e[1][5]), "+v"(e[1][6]), "+v"(e[1][7]));
        asm volatile("" : "+v"(e[2][0]), "+v"(e[2][1]), "+v"(e[2][2]), "+v"(e[2][3]), "+v"(e[2][4]), "+v"(e[2][5]), "+v"(e[2][6]), "+v"(e[2][7]),
                     "+v"(e[3][0]), "+v"(e[3][1]), "+v"(e[3][2]), "+v"(e[3][3]), "+v"(e[3][4]), "+v"(e[3][5]), "+v"(e[3][6]), "+v"(e[3][7]));
#pragma unroll
        for (int t = 1; t < T; ++t)
            asm volatile("" : "+v"(ah[t]), "+v"(al[t]));
        u32x4_b bw[4];
#define BD_PACK()                                                                                            \
        _Pragma("unroll") for (int c = 0; c < 4; ++c)                                                        \
            bw[c] = (u32x4_b){e[c][0] | (e[c][1] << 16), e[c][2] | (e[c][3] << 16), e[c][4] | (e[c][5] << 16), e[c][6] | (e[c][7] << 16)};
#define BD_MFMA(t_, c_, part_)                                                                               \
        acc[t_][c_] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_b, part_), __builtin_bit_cast(bf16x8_b, bw[c_]), acc[t_][c_], 0, 0, 0);
        BD_PACK()
        if constexpr (EXACT) {
#define BD_Z(t_, i_) ((i_) < 4 ? ah[t_][(i_) & 3] : al[t_][(i_) & 3])        /* neuron 8q + i of row bq */
            float check = 0.0f;                      // 0 * w is a NaN only for a w that is not finite
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    check = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_b, (uint32_t)bw[c][i]), (bf16x2_b){0, 0}, check, false);
            if (__any(check != check)) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
#pragma unroll 1
                    for (int g = 0; g < 4; ++g) {
                        uint32_t zr[T][4];           // neuron 8g + i of this lane's rows 4q .. 4q+3
#pragma unroll
                        for (int t = 0; t < T; ++t)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                zr[t][r] = (uint32_t)__shfl((int)BD_Z(t, i), g * 16 + 4 * q + r);
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const float w = bf16_bits_to_f32((uint32_t)__shfl((int)e[c][i], g * 16 + bq));
                            const bool bad = (__float_as_uint(w) & 0x7F800000u) == 0x7F800000u;
#pragma unroll
                            for (int t = 0; t < T; ++t)
#pragma unroll
                                for (int r = 0; r < 4; ++r)
                                    if (bad && zr[t][r] != NO_Z)
                                        acc[t][c][r] += __uint_as_float(zr[t][r]) * w;
                        }
                    }
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if ((e[c][i] & 0x7F80u) == 0x7F80u)
                            e[c][i] = (e[c][i] & 0x8000u) | 0x3F80u;
                }
                BD_PACK()
            }
            // the first, second and third eight bits of z
#pragma unroll
            for (int t = 0; t < T; ++t) {
                u32x4_b part[3];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t z[2], r[2], l[2];
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        z[k] = BD_Z(t, 2 * i + k);
                        const float f = __uint_as_float(z[k]);
                        r[k] = (z[k] & 0x7F800000u) != 0x7F800000u ? __float_as_uint(f - __uint_as_float(z[k] & 0xFFFF0000u)) : 0u;
                        l[k] = __float_as_uint(__uint_as_float(r[k]) - __uint_as_float(r[k] & 0xFFFF0000u));
                    }
                    part[0][i] = __builtin_amdgcn_perm(z[1], z[0], 0x07060302u);       // their upper halves
                    part[1][i] = __builtin_amdgcn_perm(r[1], r[0], 0x07060302u);
                    part[2][i] = __builtin_amdgcn_perm(l[1], l[0], 0x07060302u);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        BD_MFMA(t, c, part[k])
            }
#undef BD_Z
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    BD_MFMA(t, c, ah[t])
                    BD_MFMA(t, c, al[t])
                }
        }
#undef BD_PACK
#undef BD_MFMA
    }
    }
    __builtin_amdgcn_s_waitcnt(bt_vmcnt(0));                   // no LDS-DMA may outlive the loop
#undef BD_ISSUE
    // lane (column bq, row group q) holds rows 4q .. 4q+3 of every tile of the batch
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int b = t * BT_ROWS + 4 * q + i, col = c0 + c * 16 + bq;
                if (b < p.rows && col < p.d)
                    p.part[((int64_t)b * p.NR + nr) * p.d + col] = acc[t][c][i];
            }
}

// Rows with their own expert sets through the FULL block in one pass (Section 4.2: every sample picks
// its own neurons): the sets of a batch cover nearly every neuron between them (16 half-sets of a
// 14336-neuron block: all of it), so streaming the block once and dropping, per row, the neurons its
// set does not hold moves 8 times fewer bytes than streaming 16 compact blocks.  mask[g][j] collects,
// for the rows 16 g .. 16 g + 15, which of them selected neuron j.
__global__ __launch_bounds__(256) void batch_mask_zero_kernel(uint32_t *mask, int n)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j < n)
        mask[j] = 0u;
}

__global__ __launch_bounds__(256) void batch_mask_build_kernel(const int32_t *idx, int k, int n_src, uint32_t *mask)
{
    const int t = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
    if (t >= k)
        return;
    int j = idx[(int64_t)b * k + t];
    j = j < 0 ? 0 : (j >= n_src ? n_src - 1 : j);
    atomicOr(&mask[(int64_t)(b / BT_ROWS) * n_src + j], 1u << b % BT_ROWS);
}

// What the batch path would do with a shape.
struct BatchPlan {
    int T, S, W;             // tiles per pass (0: the path does not take the shape), blocks per wave, waves of the first kernel
    int NR, CS;              // ranges and column slices of the second kernel
    size_t z_units;          // floats of Z's fragments
};

static BatchPlan batch_plan_tiles(int32_t d, int32_t n, int T)
{
    BatchPlan b = {0, 0, 0, 0, 0, 0};
    const int nblk = (d + 63) / 64;
    static const int s_of[] = {2, 4, 6, 8, 10, 12, 16};
    for (int S : s_of)
        if ((nblk + S - 1) / S <= BT_WAVES) {
            b.S = S;
            break;
        }
    if (b.S == 0 || n < 64 || n > BT_MAX_N || d < 64 || d % 8 != 0 || T * b.S > (b.S == 10 ? 20 : 18))
        return b;
    b.W = (nblk + b.S - 1) / b.S;
    b.CS = (d + BT_COLS - 1) / BT_COLS;
    b.NR = 256 / b.CS;                         // as many workgroups as fit the chip at once: one more than the CUs
                                               // (d = 3072: 43 x 6 = 258) and the stragglers double the kernel's time
    if (b.NR > 64) b.NR = 64;
    const int by_range = (n + bd_range(T) - 1) / bd_range(T);
    if (b.NR < by_range) b.NR = by_range;      // a workgroup's range of Z must fit the LDS
    b.z_units = (size_t)((n + 7) / 8) * 8 * 16 * T;
    b.T = T;
    return b;
}

static size_t batch_floats(const BatchPlan &b, int32_t d, int32_t n, int32_t batch)
{
    // partial rows [batch][NR][d], the fragments, a membership word per neuron and tile
    return (((size_t)batch * b.NR * d + 63) & ~(size_t)63) + b.z_units + (size_t)b.T * n;
}

// Tiles per pass.  A pass reads all the weights, so as few passes as the registers allow (x of a pass lives in them:
// 16 T rows with T S <= 18), the rows shared out evenly.  `have` floats of workspace bound it from above: first the ranges get
// longer, down to a quarter of what fills the chip (or to what the LDS holds), then the passes get narrower (in the library's own 8 MiB:
// 64 rows of 960 x 3840 34.9 us with 28 ranges instead of 64, 48 four rows at a time; 33 rows of 704 x 12784 37.2 in one pass, 48.9 in two).
static BatchPlan batch_plan(int32_t d, int32_t n, int32_t batch, size_t have)
{
    const int tiles = (batch + BT_ROWS - 1) / BT_ROWS;
    for (int passes = 1; passes <= tiles; ++passes) {
        const int T = (tiles + passes - 1) / passes;
        if (T > BT_MAX_T)
            continue;
        BatchPlan b = batch_plan_tiles(d, n, T);
        if (!b.T)
            continue;
        const int least = std::max((n + bd_range(T) - 1) / bd_range(T), b.NR / 4);
        while (b.NR > least && batch_floats(b, d, n, batch) > have)
            --b.NR;
        if (batch_floats(b, d, n, batch) <= have)
            return b;
    }
    return BatchPlan{0, 0, 0, 0, 0, 0};
}

int decode_batch_passes(int32_t d, int32_t n, int32_t batch, size_t have)
{
    const BatchPlan b = batch_plan(d, n, batch, have);
    return b.T ? (batch + b.T * BT_ROWS - 1) / (b.T * BT_ROWS) : 0;
}

// Floats that the path wants for a shape, 0 if it does not take it (or not within `have` floats).
size_t decode_batch_floats(int32_t d, int32_t n, int32_t batch, size_t have)
{
    const BatchPlan b = batch_plan(d, n, batch, have);
    return b.T ? batch_floats(b, d, n, batch) : 0;
}

size_t index_sets_words(int32_t n_block, int32_t batch)
{
    return (size_t)((batch + BT_ROWS - 1) / BT_ROWS) * n_block;
}

// The membership words of every group of 16 rows, [groups][n_block], for callers that build them once
// per prompt (the sets do not change during generation, Section 4.2).
int launch_index_sets_build(const int32_t *idx, int32_t k, int32_t batch, int32_t n_block, uint32_t *sets, hipStream_t st)
{
    const int words = (int)index_sets_words(n_block, batch);
    hipLaunchKernelGGL(batch_mask_zero_kernel, dim3((words + 255) / 256), dim3(256), 0, st, sets, words);
    hipLaunchKernelGGL(batch_mask_build_kernel, dim3((k + 255) / 256, batch), dim3(256), 0, st, idx, k, n_block, sets);
    return check_launch("batch_mask_build_kernel");
}

// Runs both kernels for every pass; leaves part[b][NR][d] for the reduce kernel.
// n_block neurons in the block; idx (or NULL) [batch][k]: the rows' own sets inside that block;
// sets (or NULL): their membership words, else they are built here.
int launch_decode_batch_front(const DecodeJob &job, int32_t n_block, const int32_t *idx, int32_t k, const uint32_t *sets,
                              size_t have, int *NR_out, hipStream_t st)
{
    const BatchPlan pl = batch_plan(job.d, n_block, job.batch, have);
    if (pl.T == 0)
        return GRIFFIN_EUNSUPPORTED;
    *NR_out = pl.NR;
    const bool gated = job.Wg != nullptr;

    BatchParams p;
    p.Wg = job.Wg; p.W1 = job.W1; p.W2 = job.W2; p.bg = job.bg; p.b1 = job.b1;
    p.ld = job.ld; p.d = job.d; p.n = n_block; p.act = job.act;
    p.W = pl.W;
    p.P = pl.W <= 4 ? 512 : 256;               // eight waves per CU
    p.NR = pl.NR; p.CS = pl.CS;
    float *z = job.part + (((size_t)job.batch * pl.NR * job.d + 63) & ~(size_t)63);
    p.z = z;
    p.exact = !decode_whole_pieces(job.d, job.batch);
    uint32_t *mask = idx ? (uint32_t *)(z + pl.z_units) : nullptr;
    p.mask = mask;

    const int max_range = ((n_block + pl.NR - 1) / pl.NR + 7 + 31) & ~31;      // of any range, in whole steps of 32
    for (int r0 = 0; r0 < job.batch; r0 += pl.T * BT_ROWS) {
        p.rows = job.batch - r0 < pl.T * BT_ROWS ? job.batch - r0 : pl.T * BT_ROWS;
        const int T = (p.rows + BT_ROWS - 1) / BT_ROWS;                        // the last pass may have fewer tiles
        p.x = (const uint16_t *)job.x + (int64_t)r0 * job.d;
        p.part = job.part + (size_t)r0 * pl.NR * job.d;
        if (sets) {
            p.mask = sets + (size_t)(r0 / BT_ROWS) * n_block;      // built once per prompt by the caller
        } else if (idx) {
            const int rcm = launch_index_sets_build(idx + (int64_t)r0 * k, k, p.rows, n_block, mask, st);
            if (rcm != GRIFFIN_OK)
                return rcm;
        }
        // the waves of a workgroup meet as seldom as the LDS (of a CU, shared by two workgroups of up to four waves) allows
        const int group_bytes = pl.W * T * (gated ? 2 : 1) * 1024, groups = ((n_block + 7) / 8 * 4 + 8 * p.P - 1) / (8 * p.P);
        p.NB = (p.P > 256 ? 72 : 144) * 1024 / group_bytes;
        if (p.NB > groups)
            p.NB = groups;
        const size_t lds1 = (size_t)p.NB * group_bytes;
#define BT_GO(S_, T_)                                                                                          \
        case S_ * 8 + T_:                                                                                      \
            if (gated) {                                                                                       \
                RAISE_LDS_LIMIT((ff_batch_gu_kernel<true, S_, T_>), 160 * 1024)                                \
                hipLaunchKernelGGL((ff_batch_gu_kernel<true, S_, T_>), dim3(p.P), dim3(p.W * 64), lds1, st, p); \
            } else {                                                                                           \
                RAISE_LDS_LIMIT((ff_batch_gu_kernel<false, S_, T_>), 160 * 1024)                               \
                hipLaunchKernelGGL((ff_batch_gu_kernel<false, S_, T_>), dim3(p.P), dim3(p.W * 64), lds1, st, p); \
            }                                                                                                  \
            break;
        switch (pl.S * 8 + T) {
            BT_GO(2, 1) BT_GO(2, 2) BT_GO(2, 3) BT_GO(2, 4)
            BT_GO(4, 1) BT_GO(4, 2) BT_GO(4, 3) BT_GO(4, 4)
            BT_GO(6, 1) BT_GO(6, 2) BT_GO(6, 3)
            BT_GO(8, 1) BT_GO(8, 2)
            BT_GO(10, 1) BT_GO(10, 2)
            BT_GO(12, 1) BT_GO(16, 1)
        default:
            return GRIFFIN_EUNSUPPORTED;       // no plan asks for another
        }
#undef BT_GO
        int rc = check_launch("ff_batch_gu_kernel");
        if (rc != GRIFFIN_OK)
            return rc;
        const dim3 g2(pl.NR * pl.CS), b2(BT_WAVES2 * 64);
        const size_t lds2 = BD_RING + (size_t)max_range * 64 * T;
#define BD_GO2(T_, EX_)                                                                                        \
        {                                                                                                      \
            RAISE_LDS_LIMIT((ff_batch_down_kernel<T_, EX_>), 160 * 1024)                                       \
            hipLaunchKernelGGL((ff_batch_down_kernel<T_, EX_>), g2, b2, lds2, st, p);                          \
        }
#define BD_GO(T_) { if (p.exact) BD_GO2(T_, true) else BD_GO2(T_, false) }
        if (T == 1) BD_GO(1) else if (T == 2) BD_GO(2) else if (T == 3) BD_GO(3) else BD_GO(4)
#undef BD_GO2
#undef BD_GO
        rc = check_launch("ff_batch_down_kernel");
        if (rc != GRIFFIN_OK)
            return rc;
    }
    return GRIFFIN_OK;
}

}  // namespace griffin
