// The prompt product's kernel for bf16 blocks (d a multiple of 64) and its epilogue: tiles of X and of the weights go straight into
// LDS and from there to the matrix cores.  ff1.hip says what it computes and chooses how it is launched; the forms with
// an activation are compiled in ff1_silu.hip, ff1_gelu.hip and ff1_relu.hip, one file each, the plain products in ff1.hip.
#pragma once
#include "common.h"

namespace griffin {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;   // one 16-byte chunk (8 bf16)

constexpr int G_BN = 128, G_BK = 64;
constexpr int G_THREADS = 256;
// s_waitcnt immediate that waits for vmcnt <= n only (expcnt / lgkmcnt fields left at "no wait")
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// Longest row stride of Z that the usual epilogue takes: the byte offsets inside a wave's 128 rows fit 31 bits.
constexpr int64_t FF1_LDZ_MAX = 1 << 22;
static_assert((127 * FF1_LDZ_MAX + 256) * 4 < 0x7FFFFFFE, "as do those of its buffer descriptors");

struct Ff1Params {
    const void *X, *Wg, *W1, *bg, *b1;
    float *Z, *rowpart;
    uint16_t *Zb;                    // optional bf16 copy of Z [M][ldzb] for the prompt-output product, or NULL
    int64_t ldx, ldw, ldz, ldzb;
    int32_t M, F, d, nt, mt;
    int32_t splits, kt_per_split;    // ranges of the contraction (1 for the activations) and 64-wide k-tiles per range
    int32_t kt_per_sum;              // k-tiles that are summed apart and then added (FF1_SUMS_APART shapes)
    int32_t z_stream;                // Z leaves with the non-temporal hint (see launch_ff1)
    int32_t rotate;                  // each column of tiles begins at another k-tile (ff1_rotates)
    int32_t nt_row;                  // row partials of a token (nt, or those of both parts of a product on two shapes of tiles)
};


// ------------------------------------------------------------------------------------ bf16 / MFMA, direct-to-LDS
// Epilogue of the main kernel.  Its MFMAs take the weight fragment as the first operand, so the
// accumulator tiles are transposed: a lane holds ONE token (column lane & 15 of the 16x16 tile) and four consecutive
// neurons, (lane >> 4) * 4 + i.  Z is then written 16 bytes at a time and a token's sum of squares needs two lane swaps only.
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// PLAIN: the kernel serves as a plain C = A B^T with fp32 output (one range of a split contraction):
// no activation, no biases, no row sums; Z points at that range's [M][F] slab.
// One accumulator value out of its AGPR, at the point of use.  Left to itself the compiler copies all
// 256 accumulator registers into VGPRs at the end of the k loop and spills a hundred of them around
// the epilogue; the asm operand keeps each value in the accumulation file until it is wanted.
__device__ __forceinline__ float ff1_acc_read(float a)
{
    float v;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
    return v;
}

// EXTRA: 2 also knows biases and the bf16 copy of Z, 1 the copy alone, 0 neither; the lean one (most models: no FF
// biases, selection alone) does not carry those branches and registers through the epilogue.
//
// A wave's tile leaves in steps of sixteen tokens x 16 NI neurons through two private LDS patches that take turns (16 rows of
// 256 B, 16-byte chunk c of row r at c ^ r: writes and reads both spread evenly over the banks): sigma and the gating product of
// one step run while the other patch is on its way back, and a step leaves as 16-byte stores that cover whole 64 NI-byte row
// pieces (stores straight from the accumulator layout would touch 16 different rows with 64 bytes each).  Every
// LDS access here is inline asm: the next tile's first LDS-DMA loads are in flight, and an access the compiler knows about
// would wait for them (and for the Z stores).
// -> true if every wave of a tile inside the matrix has issued the usual number of stores (EPI_STORES of the kernel)
template <int ACT, bool GATED, int TI, int NI, bool PLAIN, bool EQ2W, int EXTRA, bool DUAL>
__device__ __forceinline__ bool ff1_mfma_epilogue_t(const Ff1Params &p, f32x4_t (&accU)[TI][NI], f32x4_t (&accG)[TI][NI],
                                                    uint32_t patch_lds, int m0, int n0, int tile_n)
{
    constexpr int BM = 32 * TI, BN = 32 * NI, WN = 16 * NI;   // tile; columns of a wave
    // one B matrix (the plain product, or an Eq. 2 block) over a tile twice as wide: accG = columns n0 + BN ..
    constexpr bool WIDE = (PLAIN && GATED) || EQ2W;         // two column halves to store
    constexpr bool GLU = GATED && !PLAIN && !EQ2W;          // accG is the gate (Eq. 3)
    constexpr int HV = WIDE ? 2 : 1;
    int tid = threadIdx.x;
    // what follows is worked out here, tile by tile: kept over the k loop it would cost the registers that are not there
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, l15 = lane & 15, lq = lane >> 4;
    // slabs of raw products (PLAIN) are whole rows of ldz columns, a multiple of 4: the columns past F hold repeats of
    // the last one and are never read
    const int FS = PLAIN ? (int)p.ldz : p.F;
    const bool vec = ((FS | (int32_t)p.ldz) & 3) == 0 && ((uintptr_t)p.Z & 15) == 0;
    const bool hb = EXTRA == 2 && !PLAIN && (p.b1 != nullptr || (GLU && p.bg != nullptr));
    const uint16_t *b1p = (const uint16_t *)p.b1, *bgp = (const uint16_t *)p.bg;
    const bool bias8 = (((uintptr_t)p.b1 | (uintptr_t)p.bg) & 7) == 0;       // four biases per 8-byte load
    const bool usual = vec && (!hb || bias8) && p.ldz <= FF1_LDZ_MAX;
    const uint32_t patch = patch_lds + (uint32_t)(wave * 2 * 4096);
    float sq[TI];                          // sums of squares of the lane's tokens 16 ti + l15 over its neurons
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
        sq[ti] = 0.0f;
    if (usual) {
        const uint32_t wr = patch + (uint32_t)(l15 * 256);
        // a step's 16 rows of 4 NI chunks: the lane writes NI of them, and takes numbers lane + 64 j on their way out: row rrow (of
        // the step; none if the column is past the end), byte offset vo from the step's first element
        int rrow[HV][NI];
        uint32_t rd[NI], wc[NI], vo[NI], vob[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int row = (lane + 64 * j) / (4 * NI), col = (lane + 64 * j) % (4 * NI) * 4;
#pragma unroll
            for (int h = 0; h < HV; ++h)
                rrow[h][j] = n0 + (DUAL ? 0 : h * BN) + wn * WN + col < FS ? row : 1 << 30;
            rd[j] = patch + (uint32_t)(row * 256 + ((col >> 2) ^ row) * 16);
            wc[j] = wr + (uint32_t)(((4 * j + lq) ^ l15) * 16);
            vo[j] = (uint32_t)(row * (int)p.ldz + col) * 4;
            vob[j] = (uint32_t)(row * (int)p.ldzb + col) * 2;
        }
        // biases of this lane's 4 NI columns (four consecutive ones per register pair), fetched before any store
        // of Z leaves: a load behind the stores would wait for them all
        uint2 b1w[NI], bgw[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const int c = min(n0 + wn * WN + ni * 16 + lq * 4, p.F - 4);
            b1w[ni] = (hb && b1p) ? *(const uint2 *)(b1p + c) : make_uint2(0u, 0u);
            if (EQ2W)       // the second half's b1, 128 columns further on
                bgw[ni] = (hb && b1p) ? *(const uint2 *)(b1p + min(c + BN, p.F - 4)) : make_uint2(0u, 0u);
            else
                bgw[ni] = (hb && GLU && bgp) ? *(const uint2 *)(bgp + c) : make_uint2(0u, 0u);
        }
        f32x4_t pv[NI];
// step s_: token block s_ / HV, column half s_ % HV (the second half: the second set of accumulators, 128 columns further on)
#define FF1_EPI_COMPUTE(s_)                                                                                       \
        {                                                                                                         \
            const int ti_ = (s_) / HV, half_ = (s_) % HV;                                                         \
            const int nh_ = n0 + (DUAL ? 0 : half_ * BN);                                                       \
            _Pragma("unroll") for (int ni = 0; ni < NI; ++ni)                                                      \
            {                                                                                                     \
                f32x4_t v;                                                                                        \
                _Pragma("unroll") for (int e = 0; e < 4; ++e)                                                     \
                {                                                                                                 \
                    float u = ff1_acc_read(half_ == 0 ? accU[ti_][ni][e] : accG[ti_][ni][e]);                     \
                    float gt = GLU ? ff1_acc_read(accG[ti_][ni][e]) : 0.0f;                                       \
                    if (hb) {                                                                                     \
                        const uint2 &bu = (EQ2W && half_ == 1) ? bgw[ni] : b1w[ni];                               \
                        const uint32_t wu = e < 2 ? bu.x : bu.y, wg2 = e < 2 ? bgw[ni].x : bgw[ni].y;             \
                        u += __uint_as_float((e & 1) ? (wu & 0xFFFF0000u) : (wu << 16));                          \
                        if (GLU)                                                                                  \
                            gt += __uint_as_float((e & 1) ? (wg2 & 0xFFFF0000u) : (wg2 << 16));                   \
                    }                                                                                             \
                    v[e] = PLAIN ? u : (GLU ? act_apply_t<ACT>(gt) * u : act_apply_t<ACT>(u));                    \
                }                                                                                                 \
                if (nh_ + wn * WN + ni * 16 + lq * 4 >= FS)                                                       \
                    v = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};                                                        \
                if (!PLAIN) {                                                                                     \
                    sq[ti_] = fmaf(v[0], v[0], sq[ti_]); sq[ti_] = fmaf(v[1], v[1], sq[ti_]);                     \
                    sq[ti_] = fmaf(v[2], v[2], sq[ti_]); sq[ti_] = fmaf(v[3], v[3], sq[ti_]);                     \
                }                                                                                                 \
                asm volatile("ds_write_b128 %0, %1 offset:%2" :: "v"(wc[ni]), "v"(v), "n"(((s_) & 1) * 4096) : "memory"); \
                /* keep the groups apart: left alone, the scheduler pulls the accumulator reads of all groups */  \
                /* to the front and spills a hundred registers */                                                 \
                __builtin_amdgcn_sched_barrier(0);                                                                \
            }                                                                                                     \
        }
#if defined(__HIP_DEVICE_COMPILE__)      /* the host pass has no buffer builtins */
        // the wave's rows and columns of Z (of either half) and of its bf16 copy as raw buffers
        const int64_t zrow0 = m0 + wm * (16 * TI);
        const int zcol0 = n0 + wn * WN;
        float *const z0 = p.Z + zrow0 * p.ldz + zcol0, *const z1 = z0 + (DUAL ? (int64_t)p.M * p.ldz : (int64_t)BN);
        const __amdgpu_buffer_rsrc_t zr0 = __builtin_amdgcn_make_buffer_rsrc((void *)z0, 0, 0x7FFFFFFE, 0x00020000),
                                     zr1 = __builtin_amdgcn_make_buffer_rsrc((void *)z1, 0, 0x7FFFFFFE, 0x00020000),
                                     zrb = __builtin_amdgcn_make_buffer_rsrc((void *)(p.Zb + zrow0 * p.ldzb + zcol0), 0, 0x7FFFFFFE, 0x00020000);
// Z of chunk j_ of step s_, and its bf16 copy; cache-policy bit 1 = non-temporal (the two flavours must stay two instructions)
#define FF1_Z_STORE(s_, j_)                                                                                       \
        {                                                                                                         \
            const u32x4 v_ = __builtin_bit_cast(u32x4, pv[j_]);                                                   \
            const int so_ = (s_) / HV * 16 * (int)p.ldz * 4;                                                      \
            if (p.z_stream)                                                                                       \
                __builtin_amdgcn_raw_buffer_store_b128(v_, (s_) % HV ? zr1 : zr0, vo[j_], so_, 2);                \
            else                                                                                                  \
                __builtin_amdgcn_raw_buffer_store_b128(v_, (s_) % HV ? zr1 : zr0, vo[j_], so_, 0);                \
            if (EXTRA && !PLAIN && p.Zb) {                                                                        \
                typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_;                                      \
                const u32x2_ h_ = {f32x2_to_bf16x2(pv[j_][0], pv[j_][1]), f32x2_to_bf16x2(pv[j_][2], pv[j_][3])}; \
                __builtin_amdgcn_raw_buffer_store_b64(h_, zrb, vob[j_], ((s_) / HV * 16 * (int)p.ldzb + (s_) % HV * BN) * 2, 0); \
            }                                                                                                     \
        }
#else
#define FF1_Z_STORE(s_, j_) {}
#endif
        FF1_EPI_COMPUTE(0)
#pragma unroll
        for (int s = 0; s < TI * HV; ++s) {
            // the rows of step s come back while the next step is computed (LDS accesses of a wave are performed in order)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int j = 0; j < NI; ++j)
                asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(pv[j]) : "v"(rd[j]), "n"((s & 1) * 4096) : "memory");
            if (s + 1 < TI * HV) {
                FF1_EPI_COMPUTE(s + 1)
                asm volatile("s_waitcnt lgkmcnt(%0)" :: "n"(NI) : "memory");
            } else {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
#pragma unroll
            for (int j = 0; j < NI; ++j)
                asm volatile("" : "+v"(pv[j]) :: "memory");
            const int left = p.M - (m0 + wm * (16 * TI) + (s / HV) * 16);       // rows of the matrix in this step
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                if (rrow[s % HV][j] < left)
                    FF1_Z_STORE(s, j)
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#undef FF1_Z_STORE
#undef FF1_EPI_COMPUTE
    } else {
        // rows of Z that 16-byte stores cannot take or that are too far apart, or biases that 8-byte loads cannot: straight from the
        // accumulators, 16 bytes at a time where the rows can take them.  (Rows 2^22 floats apart and more, selections, us, element by element / so /
        // with rows that the path above takes: 512 tokens of 4096 x 11008 106.7 / 103.5 / 100.1, 1024 of 4096 x 14336 245 / 233 / 220, 1000 of an Eq. 2
        // block of 4096 x 16384 163 / 153 / 142.)
#pragma unroll
        for (int ti = 0; ti < TI; ++ti) {
            const int tok = m0 + wm * (16 * TI) + ti * 16 + l15;
            const bool rowok = tok < p.M;
            float *zrow = p.Z + (int64_t)min(tok, p.M - 1) * p.ldz;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int col0 = n0 + wn * WN + ni * 16 + lq * 4;
                f32x4_t z[HV];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int col = col0 + i;
                    const int cj = min(col, p.F - 1);
                    float u = ff1_acc_read(accU[ti][ni][i]);
                    float gt = GATED ? ff1_acc_read(accG[ti][ni][i]) : 0.0f;
                    if (!PLAIN && b1p) u += bf16_bits_to_f32(b1p[cj]);
                    if (GLU && bgp) gt += bf16_bits_to_f32(bgp[cj]);
                    if (EQ2W && b1p) gt += bf16_bits_to_f32(b1p[min(col + BN, p.F - 1)]);
                    z[0][i] = PLAIN ? u : (GLU ? act_apply_t<ACT>(gt) * u : act_apply_t<ACT>(u));
                    if (WIDE)
                        z[HV - 1][i] = EQ2W ? act_apply_t<ACT>(gt) : gt;
#pragma unroll
                    for (int h = 0; h < HV; ++h)
                        if (col + h * BN < p.F) {
                            sq[ti] = fmaf(z[h][i], z[h][i], sq[ti]);
                            if (rowok && !vec)
                                zrow[col + h * BN] = z[h][i];
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (vec) {                  // F is a multiple of four: all of a lane's columns are inside, or none
#pragma unroll
                    for (int h = 0; h < HV; ++h)
                        if (rowok && col0 + h * BN < p.F)
                            *(f32x4_t *)(zrow + col0 + h * BN) = z[h];
                }
            }
        }
    }
    if (PLAIN)
        return usual;
    // row sums: the four lanes of a token by lane swaps, the two waves of a token through the patches
#pragma unroll
    for (int ti = 0; ti < TI; ++ti) {
        sq[ti] = lane_groups_sum(sq[ti]);
        asm volatile("ds_write_b32 %0, %1 offset:%2" :: "v"(patch + (uint32_t)(l15 * 4)), "v"(sq[ti]), "n"(ti * 64) : "memory");
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    static_assert(BM <= G_THREADS, "a thread per token");
    if (tid < BM) {
        float q0, q1;
        const uint32_t ra = patch_lds + (uint32_t)((tid / (16 * TI)) * 4 * 4096 + (tid % (16 * TI)) * 4);
        asm volatile("ds_read_b32 %0, %1" : "=v"(q0) : "v"(ra));
        asm volatile("ds_read_b32 %0, %1 offset:8192" : "=v"(q1) : "v"(ra));
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(q0), "+v"(q1));
        if (m0 + tid < p.M)
            p.rowpart[(int64_t)(m0 + tid) * p.nt_row + tile_n] = q0 + q1;
    }
    return usual;
}

// Main path (d a multiple of 64).  Operand tiles go from global memory straight into LDS
// (buffer_load_dwordx4 ... lds: lane l of a wave instruction fills 16-byte slot l of a 1 KB
// region; no VGPR staging, no ds_write).  A k-tile is BK = 64 elements = one whole 128-byte
// cache line per row: with half lines the other half is evicted from the 32 KB vector L1
// before the next k-tile asks for it, every line crosses the L2->L1 path twice and that path
// (64 B/clk) becomes the bound.  An instruction covers 8 rows x 128 B.  A row
// of a stage is 8 slots (128 B, half of the 256 bytes the LDS banks span), logical chunk c of
// row r in slot c ^ ((r >> 1) & 7): sixteen consecutive rows then land on sixteen different
// 16-byte bank groups, which keeps the ds_read_b128 operand fetches conflict-free (with
// c ^ (r & 7) rows two apart collide and the bank-conflict counter showed the LDS stalled for
// half of its active cycles); the swizzle is applied by choosing which global chunk each lane
// loads.  Per k-tile: two k-steps of 32 on fragments that were read one k-step ahead.  Between them, a counted
// vmcnt + one bare s_barrier say that the next k-tile has landed for every wave and that every wave has read its last
// fragment of this one; the second k-step then sends X of the k-tile two ahead into the stage just read, and the first k-step of
// the next k-tile the weights of the one three ahead of this (three stages of weights and two of X fill the LDS: 160 KB).
// Loads past the last k-tile re-read the last one into a dead stage, which keeps the loop body branch-free.  (With two stages of both the
// weights leave along with X.)
//
// What bounds it and what that decided (256 x 128 x 2 tiles, 2048 tokens of 3072 x 24576, one call after another):
//   * power.  A loop of nothing but these MFMAs on random data runs at 1.77 PFLOP/s with v_mfma_f32_32x32x16 and at 2.05
//     with v_mfma_f32_16x16x32 (2.4 with zeros, either way): hence the smaller instruction, neighbours sharing an operand.
//   * the loads' issue.  One LDS-DMA instruction per 64 clocks of MFMA and no more: two of them 416 -> 446 us
//     (without the epilogue); spread out like that they need a stage more than two to land in.
//   * 32x32x16, two stages, loads under half of the time: 502 us; this: 473 (zeros 455 -> 397).  1024 tokens of 5120 x 13824
//     254 -> 232 us, whole selections 564 -> 522, 3999 -> 3880 (4096 x 14336, 20600 tokens).
//   * the epilogue is 55 us of 473: 25 of sigma and lane work, 28 of stores that all workgroups send at about the same time.
//     (Starting the workgroups of an XCD up to 7 us apart, or letting the stores drain under one k-tile more: no faster.)
typedef __attribute__((address_space(3))) void lds_void_t;
// slot swizzle of row r (rows of every stage section start at a multiple of 16)
#define FF1_SWZ(r) (((r) >> 1) & 7)

// Tiles whose accumulators leave the registers for a second set: every kt_per_sum k-tiles the products go to partial sums, which are added
// in ascending order.  That is what ranges of d (ff1_plan) compute, without slabs and a kernel that adds them (bit for bit where a tile begins
// at k-tile 0).
#define FF1_SUMS_APART(ti_, ni_) ((ti_) * (ni_) <= 16)

// What a tile of a shape has in LDS, in 16-byte slots.  Stages: tiles of up to 128 tokens x 64 neurons, which are for little work, are bound by the
// latency of the weights and take as many as the LDS holds (40 tokens of 4096 x 11008, 64 x 64 tiles: whole selections 78 us with two
// stages, 52 with six).  Else two workgroups share a CU with 64-token tiles; from 160 tokens on two stages of X and three of the weights (the ones
// that come from HBM) fill the LDS; everything else has three of both.
template <bool GATED, int TI, int NI>
struct Ff1Stages {
    static constexpr int BM = 32 * TI, BN = 32 * NI;
    static constexpr int X_ST = BM * 8, W_ST = (GATED ? 2 : 1) * BN * 8;    // slots per stage
    static constexpr bool DEEP = TI <= 4 && NI == 2;
    static constexpr int NXS = DEEP ? 8 - (TI == 2 ? 2 : TI) : TI == 2 || TI > 4 ? 2 : 3, NWS = DEEP ? NXS : TI == 2 ? 2 : 3;
    // The epilogue's patches (32 KB) live in the last weight stage, which nothing is loaded into before the k loop of the next
    // tile; blocks with one weight section have room for patches of their own.
    static constexpr int W_BASE = NXS * X_ST, PATCH = W_BASE + (GATED ? (NWS - 1) * W_ST : NWS * W_ST), PATCH_SLOTS = 4 * 2 * 256;
    static constexpr int SLOTS = PATCH + PATCH_SLOTS > W_BASE + NWS * W_ST ? PATCH + PATCH_SLOTS : W_BASE + NWS * W_ST;
    static_assert(SLOTS * 16 <= 160 * 1024, "fits the LDS of a CU");
};

// A workgroup's tiles of one shape: of the `count` of its XCD, which are consecutive from `first` on, number `slot` and every (workgroups of
// the XCD)-th after it.
template <int ACT, bool GATED, int TI, int NI, bool PLAIN, bool EQ2W, int EXTRA, bool DUAL>
__device__ __forceinline__ void ff1_walk(const Ff1Params &p, u32x4 *lds, const int first, const int count, int slot)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass has no buffer-descriptor builtins; it only needs the launch stub
    using Stages = Ff1Stages<GATED, TI, NI>;
    constexpr int BM = 32 * TI, BN = 32 * NI, BK = 64;
    constexpr int XQ = BM / 32, WQ = BN / 32;                // 8-row regions per wave per k-tile
    constexpr int WL = (GATED ? 2 : 1) * WQ;                   // LDS-DMA instructions per wave and k-tile: XQ of X, WL of the weights
    constexpr int X_ST = Stages::X_ST, W_ST = Stages::W_ST, NXS = Stages::NXS, NWS = Stages::NWS;
    // The plain product has one B matrix: its tile is 256 columns wide and the "gate" half of the
    // machinery (LDS section, fragments, accumulators) takes columns n0 + 128 .. n0 + 255, which
    // halves the X traffic per flop exactly as the dual product does.
    // DUAL: the plain kernel over both matrices of a gated block (raw products of one range of d, two slabs per range);
    // the gate's section holds Wg again and the tile is 128 columns of both.
    constexpr bool WIDE = (PLAIN && GATED && !DUAL) || EQ2W;        // EQ2W: an Eq. 2 block (no gate) through the same machinery
    static_assert(!DUAL || (PLAIN && GATED), "DUAL is a form of the plain product");
    static_assert(!EQ2W || (GATED && !PLAIN), "the Eq. 2 wide tile uses both LDS sections and both accumulator sets");
    constexpr int TILE_N = WIDE ? 2 * BN : BN;
    constexpr int W_BASE = Stages::W_BASE, PATCH = Stages::PATCH;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // XCD-aware tile order (workgroup ids congruent mod 8 share an XCD: each XCD walks its own
    // contiguous range of tiles, its workgroups side by side); with a split contraction the ranges
    // of one tile are `ntile` ids apart.  The grid holds one workgroup per CU and every workgroup
    // walks through its tiles itself, so that the first loads of the next tile can go out before
    // the epilogue of this one (a workgroup per tile leaves the CU idle while the next one starts).
    const int ntile = p.mt * p.nt;
    // Order of the tiles: panels of PANEL_M token tiles; inside a panel the token tile runs fastest, then the
    // neuron tile.  The 32 workgroups of an XCD then work on 8 token tiles x 4 neuron tiles at any time (12
    // operand slices stream through its L2 per k-tile) instead of 32 token tiles x 1 neuron tile (33 slices)
    // when the prompt batch is long; a last panel of fewer token tiles is walked the same way.  With at most
    // PANEL_M token tiles this is the plain order "token tile fastest".
    constexpr int PANEL_M = 8;
    const int full_m = (p.mt / PANEL_M) * PANEL_M, full_tiles = full_m * p.nt;
    const int wg_per_xcd = gridDim.x >> 3;
    if (slot >= count)
        return;

    // per-tile addressing: the loader maps lane -> (row of the 8-row region, slot in the row) ->
    // global chunk (un-swizzled); byte offsets are relative to the tile's first row and fit 32 bits
    // (checked at launch).  Raw buffer descriptors (32-bit data format word of gfx9-family raw
    // buffers); every access is in range by construction, the record count is not relied upon.
    constexpr int RSRC_FLAGS = 0x00020000, RSRC_RECORDS = 0x7FFFFFFE;
    int m0, n0, tile_n, kt0, KT, rot;
    float *Zt;
    uint32_t xvo[XQ], wvo[WQ], wgvo[WQ];
    __amdgpu_buffer_rsrc_t rX, rW1, rWg;
#define FF1_TILE_ADDR(logical_)                                                                          \
    {                                                                                                    \
        int al_ = lane;                                                                                  \
        asm volatile("" : "+v"(al_));          /* nothing of this is to be kept over the k loop */       \
        const int lrow = al_ >> 3;                                                                       \
        const int split_ = (logical_) / ntile, tile_ = (logical_) % ntile;                               \
        {                                                                                                \
            const int in_full_ = tile_ < full_tiles ? 1 : 0;                                             \
            const int w_ = in_full_ ? tile_ % (PANEL_M * p.nt) : tile_ - full_tiles;                     \
            const int pm_ = in_full_ ? PANEL_M : p.mt - full_m;                                          \
            tile_n = w_ / pm_;                                                                           \
            m0 = ((in_full_ ? (tile_ / (PANEL_M * p.nt)) * PANEL_M : full_m) + w_ % pm_) * BM;           \
        }                                                                                                \
        n0 = tile_n * TILE_N;                                                                            \
        Zt = PLAIN ? p.Z + (int64_t)split_ * (DUAL ? 2 : 1) * p.M * p.ldz : p.Z;                         \
        _Pragma("unroll") for (int q = 0; q < XQ; ++q)                                                   \
            xvo[q] = __umul24(min((wave * XQ + q) * 8 + lrow, p.M - 1 - m0), (uint32_t)(p.ldx * 2)) +    \
                     (uint32_t)(((al_ & 7) ^ FF1_SWZ((wave * XQ + q) * 8 + lrow)) * 16);                 \
        _Pragma("unroll") for (int q = 0; q < WQ; ++q)                                                   \
        {                                                                                                \
            wvo[q] = __umul24(min((wave * WQ + q) * 8 + lrow, p.F - 1 - n0), (uint32_t)(p.ldw * 2)) +    \
                     (uint32_t)(((al_ & 7) ^ FF1_SWZ((wave * WQ + q) * 8 + lrow)) * 16);                 \
            wgvo[q] = WIDE ? __umul24(min(BN + (wave * WQ + q) * 8 + lrow, p.F - 1 - n0), (uint32_t)(p.ldw * 2)) +\
                             (uint32_t)(((al_ & 7) ^ FF1_SWZ((wave * WQ + q) * 8 + lrow)) * 16)          \
                           : wvo[q];                                                                     \
        }                                                                                                \
        rX = __builtin_amdgcn_make_buffer_rsrc((void *)((const uint16_t *)p.X + (int64_t)m0 * p.ldx), 0, \
                                               RSRC_RECORDS, RSRC_FLAGS);                                \
        rW1 = __builtin_amdgcn_make_buffer_rsrc((void *)((const uint16_t *)p.W1 + (int64_t)n0 * p.ldw), 0,\
                                                RSRC_RECORDS, RSRC_FLAGS);                               \
        rWg = __builtin_amdgcn_make_buffer_rsrc((void *)((const uint16_t *)((GATED && (!PLAIN || DUAL) && !EQ2W) ? p.Wg : p.W1) + (int64_t)n0 * p.ldw), 0,\
                                                RSRC_RECORDS, RSRC_FLAGS);                               \
        kt0 = split_ * p.kt_per_split;                                                                   \
        KT = min(p.kt_per_split, p.d / BK - kt0);      /* k-tiles of this range (>= 1 by construction) */\
        rot = p.rotate ? tile_n % KT : 0;                                                                 \
    }
    FF1_TILE_ADDR(first + slot)

// LDS-DMA instruction number q of the X part (0 .. XQ-1) or of the weights (0 .. WL-1: W1, then Wg) of k-tile kt_, into the stage
// at slot st_.  The weight tiles carry the non-temporal hint (each is used by one wave of tiles and then never
// again; measured 3 % faster), the X tiles, which every column of tiles re-reads, do not.
#define FF1_ROT(k_) ((k_) + rot < KT ? (k_) + rot : (k_) + rot - KT)
#define FF1_SO(kt_) ((kt0 + FF1_ROT(min((kt_), KT - 1))) * (BK * 2))
#define FF1_LOAD_X(kt_, st_, q)                                                                          \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rX, (lds_void_t *)(lds + (st_) + (wave * XQ + (q)) * 64), 16, xvo[q], FF1_SO(kt_), 0, 0);
#define FF1_LOAD_W(kt_, st_, q)                                                                          \
    {                                                                                                    \
        if ((q) < WQ)                                                                                    \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rW1, (lds_void_t *)(lds + W_BASE + (st_) + (wave * WQ + (q) % WQ) * 64), 16, \
                                                     wvo[(q) % WQ], FF1_SO(kt_), 0, 2);                  \
        else                                                                                             \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rWg, (lds_void_t *)(lds + W_BASE + (st_) + BN * 8 + (wave * WQ + (q) % WQ) * 64), 16, \
                                                     wgvo[(q) % WQ], FF1_SO(kt_), 0, 2);                 \
    }
// Operand fragments are fetched with ds_read_b128 written as inline asm: the compiler makes every
// LDS load it knows about wait for ALL LDS-DMA in flight (it cannot tell the stages apart), which
// would serialise the pipeline.  The asm reads are invisible to that logic; their completion is
// awaited explicitly (FF1_WAIT_FRAGS names the registers, so the MFMAs that use them stay behind
// it), and sched_barrier keeps the hand-made interleaving of reads, DMA issues and MFMAs.
#define FF1_DS_READ(dst, addr, off) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off))
#define FF1_BARRIER()                                                                                    \
    {                                                                                                    \
        asm volatile("" ::: "memory");                                                                   \
        __builtin_amdgcn_s_barrier();                                                                    \
        asm volatile("" ::: "memory");                                                                   \
    }
#define FF1_PIN() __builtin_amdgcn_sched_barrier(0)

    f32x4_t accU[TI][NI], accG[TI][NI];            // a wave's tile: TI blocks of sixteen tokens x NI of sixteen neurons
    constexpr bool APART = GATED && !PLAIN && FF1_SUMS_APART(TI, NI);
    f32x4_t sumU[APART ? TI : 1][APART ? NI : 1], sumG[APART ? TI : 1][APART ? NI : 1];

    const int l15 = lane & 15, lq = lane >> 4, sw = FF1_SWZ(l15);
    // LDS byte addresses of this lane's fragment rows in stage 0, per k-step of 32
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t *)lds;
    uint32_t abase[2], bbase[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const int ch = (4 * kk + lq) ^ sw;
        abase[kk] = lds0 + (uint32_t)(((wm * (16 * TI) + l15) * 8 + ch) * 16);
        bbase[kk] = lds0 + (uint32_t)((W_BASE + (wn * (16 * NI) + l15) * 8 + ch) * 16);
    }
    u32x4 fa[2][TI], f1[2][NI], fg[2][NI];
    constexpr int NREADS = TI + (GATED ? 2 : 1) * NI;
    // interleaving slots per k-step, with MPS pairs of MFMAs (up, gate) or singles each
    constexpr int NSLOTS = TI * NI < 16 ? TI * NI : TI * NI % 16 == 0 ? 16 : TI * NI % 2 == 0 ? TI * NI / 2 : TI * NI / 3, MPS = TI * NI / NSLOTS;
    static_assert(NREADS <= NSLOTS * 2 && XQ <= NSLOTS && WL <= NSLOTS && TI * NI == NSLOTS * MPS, "a k-step has a slot for everything");

// read number r (0 .. NREADS-1) of fragment set F_ (16 rows = 2048 B apart): the weights first
#define FF1_READ_ONE(F_, r, sa_, sb_)                                                          \
    {                                                                                          \
        if ((r) < NI) FF1_DS_READ(f1[F_][(r) % NI], sb_, ((r) % NI) * 2048);                   \
        else if (GATED && (r) < 2 * NI) FF1_DS_READ(fg[F_][(r) % NI], sb_, BN * 128 + ((r) % NI) * 2048); \
        else FF1_DS_READ(fa[F_][((r) - (GATED ? 2 : 1) * NI) % TI], sa_, (((r) - (GATED ? 2 : 1) * NI) % TI) * 2048); \
    }
// MFMA(s) number m (0 .. TI NI - 1) of fragment set F_: tile (ti, ni) of the up product and, gated, of the gate product; weights
// first, so the result tile is neurons x tokens.  Inline asm keeps every accumulator where it is: with the builtin the compiler, which
// has no accumulation register left to turn round in, moves some eighty of them to and fro in every k-tile.  It also sees no
// MFMA hazards then: the accumulators are written well before the first and read well after the last (FF1_MFMA_GAP), and operands
// come from the LDS behind a wait.
#define FF1_MFMA_ONE(F_, m)                                                                    \
    {                                                                                          \
        const int ti_ = (m) / NI, ni_ = (ti_ & 1) ? NI - 1 - (m) % NI : (m) % NI;              \
        if (GATED && (ti_ & 1))                                                                \
            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(accG[ti_][ni_]) : "v"(fg[F_][ni_]), "v"(fa[F_][ti_])); \
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(accU[ti_][ni_]) : "v"(f1[F_][ni_]), "v"(fa[F_][ti_])); \
        if (GATED && !(ti_ & 1))                                                               \
            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(accG[ti_][ni_]) : "v"(fg[F_][ni_]), "v"(fa[F_][ti_])); \
    }
#define FF1_MFMA_GAP() asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#define FF1_WAIT_FRAGS(F_)                                                                     \
    {                                                                                          \
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                                     \
        _Pragma("unroll") for (int n_ = 0; n_ < NI; ++n_) asm volatile("" : "+v"(f1[F_][n_])); \
        if (GATED) { _Pragma("unroll") for (int n_ = 0; n_ < NI; ++n_) asm volatile("" : "+v"(fg[F_][n_])); } \
        _Pragma("unroll") for (int t_ = 0; t_ < TI; ++t_) asm volatile("" : "+v"(fa[F_][t_])); \
    }
// one k-step: MFMAs on fragment set FM_, the reads of set FR_ (k-step KR_ of the stages at slots xs_, ws_) two a slot, and the
// loads LPS of a kind a slot: if LX_, k-tile XT_ of X into the stage at slot xd_, if LW_, k-tile WT_ of the weights into the one at wd_
#define FF1_KSTEP(FM_, FR_, xs_, ws_, KR_, LX_, XT_, xd_, LW_, WT_, wd_)                       \
    {                                                                                          \
        const uint32_t sa = abase[KR_] + (uint32_t)((xs_) * 16), sb = bbase[KR_] + (uint32_t)((ws_) * 16); \
        FF1_PIN();                                                                             \
        _Pragma("unroll") for (int m = 0; m < NSLOTS; ++m)                                     \
        {                                                                                      \
            _Pragma("unroll") for (int z_ = 0; z_ < 2; ++z_)                                   \
                if (m * 2 + z_ < NREADS)                                                       \
                    FF1_READ_ONE(FR_, m * 2 + z_, sa, sb)                                      \
            if (m * LPS < XQ && (LX_))                                                         \
            {                                                                                  \
                _Pragma("unroll") for (int z_ = 0; z_ < LPS; ++z_)                             \
                    if (m * LPS + z_ < XQ)                                                     \
                        FF1_LOAD_X(XT_, xd_, m * LPS + z_ < XQ ? m * LPS + z_ : 0)             \
            }                                                                                  \
            if (m * LPS < WL && (LW_))                                                         \
            {                                                                                  \
                _Pragma("unroll") for (int z_ = 0; z_ < LPS; ++z_)                             \
                    if (m * LPS + z_ < WL)                                                     \
                        FF1_LOAD_W(WT_, wd_, m * LPS + z_)                                     \
            }                                                                                  \
            _Pragma("unroll") for (int z_ = 0; z_ < MPS; ++z_)                                 \
                FF1_MFMA_ONE(FM_, m * MPS + z_)                                                \
            FF1_PIN();                                                                         \
        }                                                                                      \
    }

    // What a tile loads before its k loop: X of the first NXS k-tiles, the weights of the first NWS - 1; k-tile 0 first.
    constexpr int AFTER0 = (NXS - 1) * XQ + (NWS - 2) * WL;    // loads behind those of k-tile 0
    // ... and what the wait in the middle of a k-tile may leave on its way: all that was issued behind the next k-tile's
    constexpr int MID = (NXS - 2) * XQ + (NWS - 2) * WL;
    // Two stages of weights, two workgroups a CU: the first k-step is too late for the weights of the next k-tile, which are waited for
    // behind it.  They leave a k-step earlier, along with X, and those of k-tile 1 when the epilogue has left their stage; as the wait in
    // the middle is for everything, loads past the last k-tile can be left out.  With the weights in the first k-step / so (us): Eq. 2 selections, 57
    // tokens of 6144 x 16276 72.6 / 69.1, 5 of 6656 x 10384 51.8 / 50.0; outputs, 64 tokens of 5120 x 13824 47.1 / 44.6, 13 of 2560 x 7552
    // 33.5 / 30.4.
    constexpr bool PAIR = NWS == 2;
    static_assert(!PAIR || (NXS == 2 && MID == 0), "the wait in the middle is for everything");
    constexpr int LPS = PAIR ? 4 : 1;
    static_assert(AFTER0 + (PAIR ? WL : 0) <= 63 && MID <= 63, "the counter holds them");
    static_assert(NXS == NWS || NXS == NWS - 1, "the wait in the middle counts on it");
    // Global store instructions that EVERY wave issues in the epilogue's usual path on a tile that lies
    // wholly inside the matrix (NI per 16-token block and column half, plus the row sums when all four waves write them).
    // The wait for k-tile 0 of the next tile may leave that many operations outstanding, no more: a
    // wave that issued fewer stores than the wait allows would sail through before its loads landed.
    constexpr int Z_STORES = TI * NI * (WIDE || DUAL ? 2 : 1), EPI_STORES = Z_STORES + ((!PLAIN && BM == G_THREADS) ? 1 : 0);
#define FF1_FIRST_LOADS()                                                                      \
    {                                                                                          \
        _Pragma("unroll") for (int q = 0; q < XQ; ++q) FF1_LOAD_X(0, 0, q)                     \
        _Pragma("unroll") for (int q = 0; q < WL; ++q) FF1_LOAD_W(0, 0, q)                     \
        _Pragma("unroll") for (int k = 1; k < NWS - 1; ++k)                                    \
        {                                                                                      \
            if (k < NXS - 1) { _Pragma("unroll") for (int q = 0; q < XQ; ++q) FF1_LOAD_X(k, k * X_ST, q) } \
            _Pragma("unroll") for (int q = 0; q < WL; ++q) FF1_LOAD_W(k, k * W_ST, q)          \
        }                                                                                      \
        _Pragma("unroll") for (int q = 0; q < XQ; ++q) FF1_LOAD_X(NXS - 1, (NXS - 1) * X_ST, q) \
    }
    FF1_FIRST_LOADS()
    bool stores_known = false;         // the tile before was whole and took the epilogue's usual path
    for (;;) {
        // k-tile 0 has landed when only the loads behind it and (from the second tile on) the
        // epilogue's stores, all issued after it, are still outstanding
        constexpr int BEHIND = PAIR ? WL : 0, W0 = AFTER0 + BEHIND + EPI_STORES, W1 = W0 + Z_STORES;
        if (PAIR) {
#pragma unroll
            for (int q = 0; q < WL; ++q)
                FF1_LOAD_W(1, W_ST, q)
        }
        if (stores_known && EXTRA && !PLAIN && p.Zb)      // twice the Z stores (more than the counter holds: 63 is as good)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(W1 > 63 ? 63 : W1));
        else if (stores_known)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(W0 > 63 ? 63 : W0));
        else
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(AFTER0 + BEHIND));
        FF1_BARRIER()
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                accU[ti][ni] = accG[ti][ni] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
        {
            const uint32_t sa = abase[0], sb = bbase[0];
#pragma unroll
            for (int r = 0; r < NREADS; ++r)
                FF1_READ_ONE(0, r, sa, sb)
        }
        FF1_MFMA_GAP()
        int xs = 0, ws = 0, wp = (NWS - 1) * W_ST;             // stages (slots) of this k-tile, and the weights' of the one before
        int kt = 0;
        for (int ke = APART ? min(p.kt_per_sum, KT) : KT;; ke = min(ke + p.kt_per_sum, KT)) {
        for (; kt < ke; ++kt) {
            const int xn = xs == (NXS - 1) * X_ST ? 0 : xs + X_ST, wnx = ws == (NWS - 1) * W_ST ? 0 : ws + W_ST;
            FF1_WAIT_FRAGS(0)
            FF1_KSTEP(0, 1, xs, ws, 1, false, 0, 0, !PAIR, kt + NWS - 1, wp)
            FF1_WAIT_FRAGS(1)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(MID));        // tile kt+1 has landed (this wave's part)
            FF1_BARRIER()                                      // ... every wave's part; tile kt is read out
            FF1_KSTEP(1, 0, xn, wnx, 0, !PAIR || kt + NXS < KT, kt + NXS, xs, PAIR && kt + NWS < KT, kt + NWS, ws)
            wp = ws;
            ws = wnx;
            xs = xn;
        }
        if (!APART || (ke == KT && ke <= p.kt_per_sum))       // one sum
            break;
        // the sums so far; behind the last they go back to where the epilogue expects them
        FF1_MFMA_GAP()
        const bool first = ke <= p.kt_per_sum, last = ke == KT;
#pragma unroll
        for (int ti = 0; ti < (APART ? TI : 0); ++ti)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float u = ff1_acc_read(accU[ti][ni][e]), g = ff1_acc_read(accG[ti][ni][e]);
                    sumU[ti][ni][e] = first ? u : sumU[ti][ni][e] + u;
                    sumG[ti][ni][e] = first ? g : sumG[ti][ni][e] + g;
                }
                accU[ti][ni] = last ? sumU[ti][ni] : (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
                accG[ti][ni] = last ? sumG[ti][ni] : (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
            }
        FF1_MFMA_GAP()
        if (last)
            break;
        }
        FF1_MFMA_GAP()
        FF1_WAIT_FRAGS(0)                                 // the reads issued for the tile past the end
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));         // no LDS-DMA of this tile is left in flight
        FF1_BARRIER()

        // this tile's coordinates for the epilogue; then the next tile's first loads go out
        Ff1Params pt = p;
        pt.Z = Zt;
        const int m0c = m0, n0c = n0, tile_nc = tile_n;
        const bool whole = m0 + BM <= p.M && n0 + TILE_N <= p.F;
        slot += wg_per_xcd;
        const bool more = slot < count;
        if (more) {
            FF1_TILE_ADDR(first + slot)
            FF1_FIRST_LOADS()
        }
        const bool usual = ff1_mfma_epilogue_t<ACT, GATED, TI, NI, PLAIN, EQ2W, EXTRA, DUAL>(pt, accU, accG, lds0 + (uint32_t)(PATCH * 16), m0c, n0c, tile_nc);
        if (!more)
            break;
        FF1_BARRIER()              // every wave is done with its patches
        stores_known = usual && whole;
    }
#undef FF1_SO
#undef FF1_ROT
#undef FF1_LOAD_X
#undef FF1_LOAD_W
#undef FF1_MFMA_GAP
#undef FF1_TILE_ADDR
#undef FF1_FIRST_LOADS
#undef FF1_BARRIER
#undef FF1_DS_READ
#undef FF1_PIN
#undef FF1_READ_ONE
#undef FF1_MFMA_ONE
#undef FF1_WAIT_FRAGS
#undef FF1_KSTEP
#endif
}

template <int ACT, bool GATED, int TI, int NI, bool PLAIN, bool EQ2W = false, int EXTRA = 2, bool DUAL = false>
__global__ __launch_bounds__(G_THREADS) void ff1_bf16_mfma_kernel(Ff1Params p)
{
    __shared__ u32x4 lds[Ff1Stages<GATED, TI, NI>::SLOTS];
    const int nblk = p.mt * p.nt * p.splits, per_xcd = (nblk + 7) / 8, first = (int)(blockIdx.x & 7) * per_xcd;
    ff1_walk<ACT, GATED, TI, NI, PLAIN, EQ2W, EXTRA, DUAL>(p, lds, first, min(per_xcd, nblk - first), blockIdx.x >> 3);
}

// Two shapes of tiles in one launch: the neurons of `a` on the first, those of `b`, which follow them, on the second.  The tiles of both
// together are dealt out evenly over the XCDs, and the second part is walked from the other end, so that the workgroups with fewer tiles
// of the first have more of it.  Kernel medians, both builds in turn in one session (us): 1024 tokens of 5120 x 13824 on 432 tiles of 256 x 128 232 to
// 233, on 256 of them and 236 of 256 x 96 222 to 224 (with the copy of Z 249 to 251 and 246 to 247); 777 tokens on 432 of 224 x 128 202 to 203, on 192
// and 320 of 224 x 96 200 to 205; 640 tokens of 4096 x 14336 on 450 of 256 x 96 146, on 256 of 160 x 128 and 256 of 160 x 96 127 to 131.  Whole selections, in turn
// in one process: 255 / 239, 225 / 214, 169 / 146.
template <int ACT, int EXTRA, int TA, int NA, int TB, int NB>
__global__ __launch_bounds__(G_THREADS) void ff1_bf16_two_shapes_kernel(Ff1Params a, Ff1Params b)
{
    constexpr int SA = Ff1Stages<true, TA, NA>::SLOTS, SB = Ff1Stages<true, TB, NB>::SLOTS;
    __shared__ u32x4 lds[SA > SB ? SA : SB];
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int tiles_a = a.mt * a.nt, tiles = tiles_a + b.mt * b.nt;
    const int a0 = (int)((int64_t)xcd * tiles_a / 8), a1 = (int)((int64_t)(xcd + 1) * tiles_a / 8);
    const int b0 = (int)((int64_t)xcd * tiles / 8) - a0, b1 = (int)((int64_t)(xcd + 1) * tiles / 8) - a1;
    ff1_walk<ACT, true, TA, NA, false, false, EXTRA, false>(a, lds, a0, a1 - a0, slot);
    __syncthreads();              // every wave is done with its patches
    ff1_walk<ACT, true, TB, NB, false, false, EXTRA, false>(b, lds, b0, b1 - b0, (int)(gridDim.x >> 3) - 1 - slot);
}

// The whole product with its activation on this kernel, tiles of 32 ti tokens x 32 ni neurons (`wide`: an Eq. 2 block, on tiles of
// 64 ni neurons; without it the tiles of such a block are 32 ti x 128).  The caller has set p.mt and p.nt accordingly.  Nothing is launched for
// a shape that is not compiled: GRIFFIN_EUNSUPPORTED.
template <int ACT>
int launch_ff1_tiles(const Ff1Params &p, int ti, int ni, bool gated, bool wide, int grid, hipStream_t st);

// The tile shapes that are compiled: X(ti, ni, time of a round of them, 256 x 128 = 1).  ff1_tile (ff1.hip) chooses among them.
#define FF1_SHAPES(X)                                                                                           \
    X(8, 4, 1.0) X(7, 4, 0.89) X(6, 4, 0.8) X(8, 3, 0.785) X(4, 4, 0.7) X(6, 3, 0.635) X(8, 2, 0.585)       \
    X(6, 2, 0.56) X(4, 2, 0.48) X(3, 2, 0.46) X(2, 2, 0.39)

// An Eq. 2 block takes the narrow tiles in place of these.
#define FF1_SHAPE_EQ2(ti_, ni_) ((ni_) > 2 || (ti_) == 2)

#define FF1_GO(...) hipLaunchKernelGGL((ff1_bf16_mfma_kernel<ACT, __VA_ARGS__>), dim3(grid), dim3(G_THREADS), 0, st, p)
#define FF1_TILES_CASE(TI_, NI_, COST_)                                                                         \
    if (ti == TI_ && ni == NI_) {                                                                               \
        if (!gated) {                                                                                           \
            if constexpr (!FF1_SHAPE_EQ2(TI_, NI_)) return GRIFFIN_EUNSUPPORTED;                                \
            else FF1_GO(true, TI_, NI_, false, true);                                                           \
        } else if (p.b1 || p.bg) {                                                                              \
            FF1_GO(true, TI_, NI_, false);                                                                      \
        } else {                                                                                                \
            if constexpr (NI_ != 2)                                                                             \
                if (!p.Zb) {                                                                                    \
                    FF1_GO(true, TI_, NI_, false, false, 0);                                                    \
                    return GRIFFIN_OK;                                                                          \
                }                                                                                               \
            FF1_GO(true, TI_, NI_, false, false, 1);                                                            \
        }                                                                                                       \
        return GRIFFIN_OK;                                                                                      \
    }
#define FF1_TILES_OF(ACT_)                                                                                      \
    template <>                                                                                                 \
    int launch_ff1_tiles<ACT_>(const Ff1Params &p, int ti, int ni, bool gated, bool wide, int grid, hipStream_t st) \
    {                                                                                                           \
        constexpr int ACT = ACT_;                                                                               \
        if (!gated && !wide) {                                                                                  \
            if (ti == 8 && ni == 4) FF1_GO(false, 8, 4, false);                                                 \
            else if (ti == 4 && ni == 4) FF1_GO(false, 4, 4, false);                                            \
            else return GRIFFIN_EUNSUPPORTED;                                                                   \
            return GRIFFIN_OK;                                                                                  \
        }                                                                                                       \
        FF1_SHAPES(FF1_TILES_CASE)                                                                              \
        return GRIFFIN_EUNSUPPORTED;                                                                            \
    }

// The product of an Eq. 3 block without biases on tiles of 32 ti tokens x 128 neurons (a) and x 96 neurons (b), in one launch.
template <int ACT>
int launch_ff1_two_shapes(const Ff1Params &a, const Ff1Params &b, int ti, int grid, hipStream_t st);

// The heights that are compiled: X(ti, time of a round of 128-neuron tiles, of 96-neuron tiles; 256 x 128 = 1)
#define FF1_TWO_SHAPES(X) X(8, 1.0, 0.78) X(7, 0.905, 0.71) X(6, 0.8, 0.63) X(5, 0.71, 0.57)
#define FF1_TWO_CASE(TI_, WIDE_, NARROW_)                                                                       \
    if (ti == TI_) {                                                                                            \
        if (a.Zb) hipLaunchKernelGGL((ff1_bf16_two_shapes_kernel<ACT, 1, TI_, 4, TI_, 3>), dim3(grid), dim3(G_THREADS), 0, st, a, b); \
        else hipLaunchKernelGGL((ff1_bf16_two_shapes_kernel<ACT, 0, TI_, 4, TI_, 3>), dim3(grid), dim3(G_THREADS), 0, st, a, b); \
        return GRIFFIN_OK;                                                                                      \
    }
#define FF1_TWO_OF(ACT_)                                                                                        \
    template <>                                                                                                 \
    int launch_ff1_two_shapes<ACT_>(const Ff1Params &a, const Ff1Params &b, int ti, int grid, hipStream_t st)   \
    {                                                                                                           \
        constexpr int ACT = ACT_;                                                                               \
        FF1_TWO_SHAPES(FF1_TWO_CASE)                                                                            \
        return GRIFFIN_EUNSUPPORTED;                                                                            \
    }

}  // namespace griffin
