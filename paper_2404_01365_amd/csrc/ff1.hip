// Prompt phase, first half: the FF activations of every prompt token (Section 3, Eq. 3 applied
// row-wise; Eq. 2 when there is no gate),
//     Z = sigma(X Wg^T + bg) * (X W1^T + b1),
// together with one sum-of-squares partial per (token row, column tile) from which the row
// norms of Section 4.1 are finished elsewhere.
//
// bf16: a dense contraction, so it runs on the matrix cores.  One workgroup (4 wavefronts, 2x2)
// owns a 256-token (128 for short prompts) x 128-neuron tile of BOTH products: the X tile is
// staged once in LDS and feeds two sets of v_mfma_f32_16x16x32_bf16 accumulators (gate and up),
// so the epilogue finds g_ij and u_ij in the same lane and applies sigma, the gating product,
// the store of Z and the row sum-of-squares without another pass.  Workgroup ids are remapped so
// that each XCD (ids congruent mod 8 land on the same XCD) walks a contiguous range of tiles and
// reuses W tiles in its own L2.  The main kernel loads tiles straight into LDS; a register-staged
// variant takes the shapes it cannot (d not a multiple of 64).
//
// fp32 blocks: f32.hip.
#include "common.h"

#include <atomic>

namespace griffin {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;   // one 16-byte chunk (8 bf16)

constexpr int G_BN = 128, G_BK = 64;
constexpr int G_THREADS = 256;
// s_waitcnt immediate that waits for vmcnt <= n only (expcnt / lgkmcnt fields left at "no wait")
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

struct Ff1Params {
    const void *X, *Wg, *W1, *bg, *b1;
    float *Z, *rowpart;
    uint16_t *Zb;                    // optional bf16 copy of Z [M][ldzb] for the prompt-output product, or NULL
    int64_t ldx, ldw, ldz, ldzb;
    int32_t M, F, d, nt, mt;
    int32_t splits, kt_per_split;    // ranges of the contraction (1 for the activations) and 64-wide k-tiles per range
    int32_t z_stream;                // Z leaves with the non-temporal hint (see launch_ff1)
};

// Epilogue shared by the MFMA kernels: sigma, gating, store of Z, row sums of z^2.
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
    const bool usual = vec && (!hb || bias8) && p.ldz <= (1 << 20);         // (32-bit byte offsets inside a tile)
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
        // rows of Z that 16-byte stores cannot take, or biases that 8-byte loads cannot: element by element
#pragma unroll
        for (int ti = 0; ti < TI; ++ti) {
            const int tok = m0 + wm * (16 * TI) + ti * 16 + l15;
            const bool rowok = tok < p.M;
            float *zrow = p.Z + (int64_t)min(tok, p.M - 1) * p.ldz;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int col = n0 + wn * WN + ni * 16 + lq * 4 + i;
                    const int cj = min(col, p.F - 1);
                    float u = ff1_acc_read(accU[ti][ni][i]);
                    float gt = GATED ? ff1_acc_read(accG[ti][ni][i]) : 0.0f;
                    if (!PLAIN && b1p) u += bf16_bits_to_f32(b1p[cj]);
                    if (GLU && bgp) gt += bf16_bits_to_f32(bgp[cj]);
                    if (EQ2W && b1p) gt += bf16_bits_to_f32(b1p[min(col + BN, p.F - 1)]);
                    const float z = PLAIN ? u : (GLU ? act_apply_t<ACT>(gt) * u : act_apply_t<ACT>(u));
                    if (col < p.F) {
                        sq[ti] = fmaf(z, z, sq[ti]);
                        if (rowok)
                            zrow[col] = z;
                    }
                    if (WIDE && col + BN < p.F) {
                        const float z2 = EQ2W ? act_apply_t<ACT>(gt) : gt;
                        sq[ti] = fmaf(z2, z2, sq[ti]);
                        if (rowok)
                            zrow[col + BN] = z2;
                    }
                    __builtin_amdgcn_sched_barrier(0);
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
            p.rowpart[(int64_t)(m0 + tid) * p.nt + tile_n] = q0 + q1;
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
// Loads past the last k-tile re-read the last one into a dead stage, which keeps the loop body branch-free.
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

template <int ACT, bool GATED, int TI, int NI, bool PLAIN, bool EQ2W = false, int EXTRA = 2, bool DUAL = false>
__global__ __launch_bounds__(G_THREADS) void ff1_bf16_mfma_kernel(Ff1Params p)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass has no buffer-descriptor builtins; it only needs the launch stub
    constexpr int BM = 32 * TI, BN = 32 * NI, BK = 64;
    constexpr int XQ = BM / 32, WQ = BN / 32;                // 8-row regions per wave per k-tile
    constexpr int WL = (GATED ? 2 : 1) * WQ;                   // LDS-DMA instructions per wave and k-tile: XQ of X, WL of the weights
    constexpr int X_ST = BM * 8, W_ST = (GATED ? 2 : 1) * BN * 8;    // 16-byte slots per stage
    // Stages: two workgroups share a CU with 64-token tiles; 256-token tiles of two weight sections fill the LDS with two stages of X
    // and three of the weights (the ones that come from HBM); everything else has three of both.
    constexpr int NXS = TI == 2 || TI > 4 ? 2 : 3, NWS = TI == 2 ? 2 : 3;
    // The plain product has one B matrix: its tile is 256 columns wide and the "gate" half of the
    // machinery (LDS section, fragments, accumulators) takes columns n0 + 128 .. n0 + 255, which
    // halves the X traffic per flop exactly as the dual product does.
    // DUAL: the plain kernel over both matrices of a gated block (raw products of one range of d, two slabs per range);
    // the gate's section holds Wg again and the tile is 128 columns of both.
    constexpr bool WIDE = (PLAIN && GATED && !DUAL) || EQ2W;        // EQ2W: an Eq. 2 block (no gate) through the same machinery
    static_assert(!DUAL || (PLAIN && GATED), "DUAL is a form of the plain product");
    static_assert(!EQ2W || (GATED && !PLAIN), "the Eq. 2 wide tile uses both LDS sections and both accumulator sets");
    constexpr int TILE_N = WIDE ? 2 * BN : BN;
    // The epilogue's patches (32 KB) live in the last weight stage, which nothing is loaded into before the k loop of the next
    // tile; blocks with one weight section have room for patches of their own.
    constexpr int W_BASE = NXS * X_ST, PATCH = W_BASE + (GATED ? (NWS - 1) * W_ST : NWS * W_ST), PATCH_SLOTS = 4 * 2 * 256;
    constexpr int LDS_SLOTS = PATCH + PATCH_SLOTS > W_BASE + NWS * W_ST ? PATCH + PATCH_SLOTS : W_BASE + NWS * W_ST;
    static_assert(LDS_SLOTS * 16 <= 160 * 1024, "fits the LDS of a CU");
    __shared__ u32x4 lds[LDS_SLOTS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // XCD-aware tile order (workgroup ids congruent mod 8 share an XCD: each XCD walks its own
    // contiguous range of tiles, its workgroups side by side); with a split contraction the ranges
    // of one tile are `ntile` ids apart.  The grid holds one workgroup per CU and every workgroup
    // walks through its tiles itself, so that the first loads of the next tile can go out before
    // the epilogue of this one (a workgroup per tile leaves the CU idle while the next one starts).
    const int ntile = p.mt * p.nt, nblk = ntile * p.splits;
    // Order of the tiles: panels of PANEL_M token tiles; inside a panel the token tile runs fastest, then the
    // neuron tile.  The 32 workgroups of an XCD then work on 8 token tiles x 4 neuron tiles at any time (12
    // operand slices stream through its L2 per k-tile) instead of 32 token tiles x 1 neuron tile (33 slices)
    // when the prompt batch is long; a last panel of fewer token tiles is walked the same way.  With at most
    // PANEL_M token tiles this is the plain order "token tile fastest".
    constexpr int PANEL_M = 8;
    const int full_m = (p.mt / PANEL_M) * PANEL_M, full_tiles = full_m * p.nt;
    const int per_xcd = (nblk + 7) / 8;
    const int wg_per_xcd = gridDim.x >> 3;
    int slot = blockIdx.x >> 3;
    if (slot >= per_xcd || (int)(blockIdx.x & 7) * per_xcd + slot >= nblk)
        return;

    // per-tile addressing: the loader maps lane -> (row of the 8-row region, slot in the row) ->
    // global chunk (un-swizzled); byte offsets are relative to the tile's first row and fit 32 bits
    // (checked at launch).  Raw buffer descriptors (32-bit data format word of gfx9-family raw
    // buffers); every access is in range by construction, the record count is not relied upon.
    constexpr int RSRC_FLAGS = 0x00020000, RSRC_RECORDS = 0x7FFFFFFE;
    int m0, n0, tile_n, kt0, KT;
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
    }
    FF1_TILE_ADDR((int)(blockIdx.x & 7) * per_xcd + slot)

// LDS-DMA instruction number q of the X part (0 .. XQ-1) or of the weights (0 .. WL-1: W1, then Wg) of k-tile kt_, into the stage
// at slot st_.  The weight tiles carry the non-temporal hint (each is used by one wave of tiles and then never
// again; measured 3 % faster), the X tiles, which every column of tiles re-reads, do not.
#define FF1_SO(kt_) ((kt0 + min((kt_), KT - 1)) * (BK * 2))
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
    constexpr int NSLOTS = TI * NI < 16 ? TI * NI : TI * NI % 16 == 0 ? 16 : 12;          // interleaving slots per k-step ...
    constexpr int MPS = TI * NI / NSLOTS;                      // ... with so many pairs of MFMAs (up, gate) or singles each
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
// loads one a slot: LX_ a k-tile of X, else one of the weights, LT_ into the stage at slot ls_
#define FF1_KSTEP(FM_, FR_, xs_, ws_, KR_, LX_, LT_, ls_)                                      \
    {                                                                                          \
        const uint32_t sa = abase[KR_] + (uint32_t)((xs_) * 16), sb = bbase[KR_] + (uint32_t)((ws_) * 16); \
        FF1_PIN();                                                                             \
        _Pragma("unroll") for (int m = 0; m < NSLOTS; ++m)                                     \
        {                                                                                      \
            _Pragma("unroll") for (int z_ = 0; z_ < 2; ++z_)                                   \
                if (m * 2 + z_ < NREADS)                                                       \
                    FF1_READ_ONE(FR_, m * 2 + z_, sa, sb)                                      \
            if ((LX_) && m < XQ)                                                               \
                FF1_LOAD_X(LT_, ls_, m < XQ ? m : 0)                                           \
            if (!(LX_) && m < WL)                                                              \
                FF1_LOAD_W(LT_, ls_, m)                                                        \
            _Pragma("unroll") for (int z_ = 0; z_ < MPS; ++z_)                                 \
                FF1_MFMA_ONE(FM_, m * MPS + z_)                                                \
            FF1_PIN();                                                                         \
        }                                                                                      \
    }

    // What a tile loads before its k loop: X of the first NXS k-tiles, the weights of the first NWS - 1; k-tile 0 first.
    constexpr int AFTER0 = (NXS - 1) * XQ + (NWS - 2) * WL;    // loads behind those of k-tile 0
    // ... and what of it the wait in the middle of a k-tile may leave on its way: the last X (three stages) and weights (three)
    constexpr int MID = (NXS == 3 ? XQ : 0) + (NWS == 3 ? WL : 0);
    static_assert(NXS <= NWS, "the wait in the middle counts on it");
    // Global store instructions that EVERY wave issues in the epilogue's usual path on a tile that lies
    // wholly inside the matrix (NI per 16-token block and column half, plus the row sums when all four waves write them).
    // The wait for k-tile 0 of the next tile may leave that many operations outstanding, no more: a
    // wave that issued fewer stores than the wait allows would sail through before its loads landed.
    constexpr int Z_STORES = TI * NI * (WIDE || DUAL ? 2 : 1), EPI_STORES = Z_STORES + ((!PLAIN && BM == G_THREADS) ? 1 : 0);
#define FF1_FIRST_LOADS()                                                                      \
    {                                                                                          \
        _Pragma("unroll") for (int q = 0; q < XQ; ++q) FF1_LOAD_X(0, 0, q)                     \
        _Pragma("unroll") for (int q = 0; q < WL; ++q) FF1_LOAD_W(0, 0, q)                     \
        if (NXS == 3) { _Pragma("unroll") for (int q = 0; q < XQ; ++q) FF1_LOAD_X(1, X_ST, q) } \
        if (NWS == 3) { _Pragma("unroll") for (int q = 0; q < WL; ++q) FF1_LOAD_W(1, W_ST, q) } \
        _Pragma("unroll") for (int q = 0; q < XQ; ++q) FF1_LOAD_X(NXS - 1, (NXS - 1) * X_ST, q) \
    }
    FF1_FIRST_LOADS()
    bool stores_known = false;         // the tile before was whole and took the epilogue's usual path
    for (;;) {
        // k-tile 0 has landed when only the loads behind it and (from the second tile on) the
        // epilogue's stores, all issued after it, are still outstanding
        constexpr int W0 = AFTER0 + EPI_STORES, W1 = W0 + Z_STORES;
        if (stores_known && EXTRA && !PLAIN && p.Zb)      // twice the Z stores (more than the counter holds: 63 is as good)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(W1 > 63 ? 63 : W1));
        else if (stores_known)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(W0 > 63 ? 63 : W0));
        else
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(AFTER0));
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
        for (int kt = 0; kt < KT; ++kt) {
            const int xn = xs == (NXS - 1) * X_ST ? 0 : xs + X_ST, wnx = ws == (NWS - 1) * W_ST ? 0 : ws + W_ST;
            FF1_WAIT_FRAGS(0)
            FF1_KSTEP(0, 1, xs, ws, 1, false, kt + NWS - 1, wp)
            FF1_WAIT_FRAGS(1)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(MID));        // tile kt+1 has landed (this wave's part)
            FF1_BARRIER()                                      // ... every wave's part; tile kt is read out
            FF1_KSTEP(1, 0, xn, wnx, 0, true, kt + NXS, xs)
            wp = ws;
            ws = wnx;
            xs = xn;
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
        const int logical_n = (int)(blockIdx.x & 7) * per_xcd + slot;
        const bool more = slot < per_xcd && logical_n < nblk;
        if (more) {
            FF1_TILE_ADDR(logical_n)
            FF1_FIRST_LOADS()
        }
        const bool usual = ff1_mfma_epilogue_t<ACT, GATED, TI, NI, PLAIN, EQ2W, EXTRA, DUAL>(pt, accU, accG, lds0 + (uint32_t)(PATCH * 16), m0c, n0c, tile_nc);
        if (!more)
            break;
        FF1_BARRIER()              // every wave is done with its patches
        stores_known = usual && whole;
    }
#undef FF1_SO
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

struct Ff1Plan {
    int splits, per;         // ranges of d, k-tiles per range; 1 range: the epilogue of the product does it all
    int64_t ldu;             // columns of a slab's row
};

// How many ranges: the cheapest by a cost in microseconds, from (measured) the time of a k-tile on a CU with its item's
// fixed part in k-tiles, the weights at the rate the loop draws them from HBM, the slabs written and read again, and the
// second kernel:
//   * the whole product: a k-tile 1.15 us (256 tokens; 1.05 with up to 128; an Eq. 2 block's 128-column tiles 0.95 / 0.8), 8 (3)
//     k-tiles of prologue and epilogue;
//   * in ranges: the same without sigma in the epilogue (5, 3); up to 64 tokens 1.0 us, 1.25 us where two workgroups share a CU.
// Whole selections of a 4096 x 11008 block, in one range / in 2, 3, 4, 5, 8 ranges (us): 40 tokens 96 / 70, 69, 64, 65, 70;
// 128 tokens 97 / 75, 97, 87, 84, 102; 256 tokens 111 / 88, 120, 114, 112, 138; 512 tokens 115 / 152, 178, ...; of a 2048 x 8192
// block: 40 tokens 58 / 45, 42, 41, 44, 46; 256 tokens 70 / 60, 58, 59, 83, 89; of a 8192 x 8192 Eq. 2 block: 40 tokens
// 127 / 92, 73, 64, 58, 52; 512 tokens 151 / 120, 101, 107, 134, 125.
static Ff1Plan ff1_plan(const griffin_layer &L, int64_t M)
{
    const int KT = L.d / 64;
    Ff1Plan pl = {1, KT, ((int64_t)L.n + 3) & ~(int64_t)3};
    if (L.dtype != GRIFFIN_BF16 || L.d % 64 != 0 || L.ld > (1 << 21) || M < 1 || M > 2048)
        return pl;
    const bool gated = L.Wg != nullptr;
    const int64_t mt = M > 128 ? (M + 255) / 256 : 1;
    const int64_t n128 = mt * ((L.n + G_BN - 1) / G_BN), n256 = mt * ((L.n + 2 * G_BN - 1) / (2 * G_BN));
    const int fix_whole = M > 128 ? 8 : 3, fix_raw = M > 128 ? 5 : 3;
    const double kt_us = M > 128 ? 1.15 : 1.05, kt_narrow_us = M > 128 ? 0.95 : 0.8;
    double best = (double)((n128 + 255) / 256) * (KT + fix_whole) * (gated ? kt_us : kt_narrow_us);
    if (!gated) {
        const double wide = (double)((n256 + 255) / 256) * (KT + fix_whole) * kt_us;
        best = wide < best ? wide : best;
    }
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
            pl.splits = used;
            pl.per = per;
        }
    }
    return pl;
}

size_t ff1_slab_bytes(const griffin_layer &L, int64_t M)
{
    const Ff1Plan pl = ff1_plan(L, M);
    return pl.splits > 1 ? (size_t)pl.splits * (L.Wg ? 2 : 1) * M * pl.ldu * sizeof(float) : 0;
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

template <int ACT, int MI>
static void launch_mfma(const Ff1Params &p, bool gated, bool wide, hipStream_t st)
{
    const int nblk = p.mt * p.nt;
    dim3 grid(ff1_grid(nblk)), block(G_THREADS);
    dim3 grid_all(((nblk + 7) / 8) * 8);           // the register-staged kernel takes one tile per workgroup
    // the direct-to-LDS kernel wants whole 64-element k-tiles and 32-bit byte offsets inside a tile
    const bool ktail = p.d % 64 != 0 || p.ldx > (1 << 21) || p.ldw > (1 << 21);
    if (gated) {
        if (ktail) hipLaunchKernelGGL((ff1_bf16_mfma_staged_kernel<ACT, true, MI, true>), grid_all, block, 0, st, p);
        else if (p.b1 || p.bg) hipLaunchKernelGGL((ff1_bf16_mfma_kernel<ACT, true, 2 * MI, 4, false>), grid, block, 0, st, p);
        else if (p.Zb) hipLaunchKernelGGL((ff1_bf16_mfma_kernel<ACT, true, 2 * MI, 4, false, false, 1>), grid, block, 0, st, p);
        else hipLaunchKernelGGL((ff1_bf16_mfma_kernel<ACT, true, 2 * MI, 4, false, false, 0>), grid, block, 0, st, p);
    } else {
        if (ktail) hipLaunchKernelGGL((ff1_bf16_mfma_staged_kernel<ACT, false, MI, true>), grid_all, block, 0, st, p);
        else if (wide) hipLaunchKernelGGL((ff1_bf16_mfma_kernel<ACT, true, 2 * MI, 4, false, true>), grid, block, 0, st, p);   // 256-column tiles
        else hipLaunchKernelGGL((ff1_bf16_mfma_kernel<ACT, false, 2 * MI, 4, false>), grid, block, 0, st, p);
    }
}

template <int MI>
static void launch_mfma_act(const Ff1Params &p, int act, bool gated, bool wide, hipStream_t st)
{
    switch (act) {
    case GRIFFIN_ACT_SILU: launch_mfma<GRIFFIN_ACT_SILU, MI>(p, gated, wide, st); break;
    case GRIFFIN_ACT_GELU_TANH: launch_mfma<GRIFFIN_ACT_GELU_TANH, MI>(p, gated, wide, st); break;
    default: launch_mfma<GRIFFIN_ACT_RELU, MI>(p, gated, wide, st); break;
    }
}

// Will the first GEMM's own epilogue leave a bf16 copy of Z beside the fp32 one?  Only the direct-to-LDS
// kernel's usual store path does (bf16 block, d in whole k-tiles, 16-byte aligned rows of Z, biases 8-byte aligned).
bool ff1_can_write_zb(const griffin_layer &L, int64_t ldx, const float *Z, int64_t ldz)
{
    const bool ktail = L.d % 64 != 0 || ldx > (1 << 21) || L.ld > (1 << 21);
    const bool vec = ((L.n | (int32_t)ldz) & 3) == 0 && ((uintptr_t)Z & 15) == 0;
    const bool bias8 = (((uintptr_t)L.b1 | (uintptr_t)L.bg) & 7) == 0;
    return L.dtype == GRIFFIN_BF16 && !ktail && vec && bias8 && ldz <= (1 << 20);
}

int launch_ff1(const griffin_layer &L, const void *X, int64_t ldx, int64_t M, float *Z, int64_t ldz,
               float *rowpart, int32_t *nt_out, hipStream_t st, uint16_t *Zb, int64_t ldzb, float *slabs)
{
    Ff1Params p;
    p.X = X; p.Wg = L.Wg; p.W1 = L.W1; p.bg = L.bg; p.b1 = L.b1;
    p.Z = Z; p.rowpart = rowpart;
    p.Zb = (Zb && ff1_can_write_zb(L, ldx, Z, ldz)) ? Zb : nullptr;
    p.ldzb = ldzb;
    p.ldx = ldx; p.ldw = L.ld; p.ldz = ldz;
    p.M = (int32_t)M; p.F = L.n; p.d = L.d;
    p.splits = 1; p.kt_per_split = L.d / 64;
    // Z is read again at once by the statistic kernel.  While it fits the 256 MB Infinity Cache, plain stores leave it
    // there for that kernel; a Z several times that size is better sent past the caches (measured, statistic kernel
    // after plain / non-temporal stores: 201 MB of Z 38.3 / 44.6 us, 57 MB 14.5 / 16.4 us, 1.18 GB 284 / 243 us; the
    // product itself takes the same time either way).
    p.z_stream = ((int64_t)M * L.n * 4 > ((int64_t)384 << 20) && ldz <= (1 << 20)) ? 1 : 0;   // (32-bit byte offsets inside a tile)
    p.nt = ff1_ntiles(L);
    const bool gated = L.Wg != nullptr;
    // An Eq. 2 block on the direct-to-LDS kernel takes 256-column tiles (one row-sum partial per tile) when that
    // is the faster way to fill the chip: a 128-column tile of one product is bound by the L2->L1 path (~1400
    // clocks per k-tile), a 256-column tile by the matrix cores (~2550), and either comes in rounds of one tile per CU.
    bool wide = false;
    if (L.dtype == GRIFFIN_BF16 && !gated && !(L.d % 64 != 0 || ldx > (1 << 21) || L.ld > (1 << 21))) {
        const int64_t mt = M > 128 ? (M + 255) / 256 : (M + 127) / 128;
        const int64_t tn = mt * p.nt, tw = mt * ((L.n + 2 * G_BN - 1) / (2 * G_BN));
        wide = ((tw + 255) / 256) * 2550 < ((tn + 255) / 256) * 1400;
        if (wide)
            p.nt = (L.n + 2 * G_BN - 1) / (2 * G_BN);
    }
    const Ff1Plan pl = ff1_plan(L, M);
    if (slabs && pl.splits > 1 && ldx <= (1 << 21)) {
        const int nb = (L.n + ACT_COLS - 1) / ACT_COLS;
        *nt_out = nb;
        int rc;
        if (gated) {
            p.Z = slabs; p.ldz = pl.ldu; p.Zb = nullptr; p.z_stream = 0;
            p.splits = pl.splits; p.kt_per_split = pl.per;
            p.mt = (int32_t)(M > 128 ? (M + 255) / 256 : 1);
            const dim3 grid(ff1_grid(p.mt * p.nt * pl.splits, M <= 64 ? 2 : 1)), block(G_THREADS);
            if (M <= 64)
                hipLaunchKernelGGL((ff1_bf16_mfma_kernel<GRIFFIN_ACT_RELU, true, 2, 4, true, false, 2, true>), grid, block, 0, st, p);
            else if (M > 128)
                hipLaunchKernelGGL((ff1_bf16_mfma_kernel<GRIFFIN_ACT_RELU, true, 8, 4, true, false, 2, true>), grid, block, 0, st, p);
            else
                hipLaunchKernelGGL((ff1_bf16_mfma_kernel<GRIFFIN_ACT_RELU, true, 4, 4, true, false, 2, true>), grid, block, 0, st, p);
            rc = check_launch("ff1_bf16_mfma_kernel");
        } else {
            rc = launch_gemm_nt_partials(X, ldx, L.W1, L.ld, M, L.n, L.d, pl.splits, pl.per, slabs, pl.ldu, st);
        }
        if (rc != GRIFFIN_OK)
            return rc;
        Ff1ActParams a;
        a.U = slabs; a.bg = L.bg; a.b1 = L.b1; a.Z = Z; a.rowpart = rowpart;
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
    *nt_out = p.nt;
    if (M == 0)
        return GRIFFIN_OK;
    if (L.dtype == GRIFFIN_BF16) {
        // 256-token tiles halve the LDS traffic per flop; short prompts keep 128
        if (M > 128) {
            p.mt = (int32_t)((M + 255) / 256);
            launch_mfma_act<4>(p, L.act, gated, wide, st);
        } else {
            p.mt = (int32_t)((M + 127) / 128);
            launch_mfma_act<2>(p, L.act, gated, wide, st);
        }
        return check_launch("ff1_bf16_mfma_kernel");
    }
    return launch_f32_ff1(L, X, ldx, M, Z, ldz, rowpart, st);
}

// C[s] = A B^T over the s-th range of the contraction, fp32, for s = 0 .. splits-1, on the
// direct-to-LDS kernel: A [M][K] and B [N][K] bf16 with K a multiple of 64, C [splits][M][ldc], ldc a multiple of 4.
// Used by the prompt-output GEMM (Section 5.1) on a bf16 copy of Z.
bool gemm_nt_partials_ok(int64_t M, int32_t N, int32_t K, int64_t lda, int64_t ldb)
{
    return M >= 1 && M <= (1 << 30) && K % 64 == 0 && N % 4 == 0 && lda % 8 == 0 && ldb % 8 == 0 &&
           lda <= (1 << 21) && ldb <= (1 << 21);
}

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
    Ff1Params p;
    p.X = A; p.Wg = nullptr; p.W1 = B; p.bg = nullptr; p.b1 = nullptr;
    p.Z = C; p.rowpart = nullptr;
    p.Zb = nullptr; p.ldzb = 0;
    p.ldx = lda; p.ldw = ldb; p.ldz = ldc;
    p.M = (int32_t)M; p.F = N; p.d = K;
    p.splits = splits; p.kt_per_split = kt_per_split;
    p.z_stream = 0;
    p.nt = (N + 2 * G_BN - 1) / (2 * G_BN);        // 256-column tiles: both sets of accumulators hold columns of B
    if (M > 128) {
        p.mt = (int32_t)((M + 255) / 256);
        const int nblk = p.mt * p.nt * splits;
        hipLaunchKernelGGL((ff1_bf16_mfma_kernel<GRIFFIN_ACT_RELU, true, 8, 4, true>), dim3(ff1_grid(nblk)), dim3(G_THREADS), 0, st, p);
    } else if (M <= 64) {
        p.mt = 1;
        hipLaunchKernelGGL((ff1_bf16_mfma_kernel<GRIFFIN_ACT_RELU, true, 2, 4, true>), dim3(ff1_grid(p.nt * splits, 2)), dim3(G_THREADS), 0, st, p);
    } else {
        p.mt = (int32_t)((M + 127) / 128);
        const int nblk = p.mt * p.nt * splits;
        hipLaunchKernelGGL((ff1_bf16_mfma_kernel<GRIFFIN_ACT_RELU, true, 4, 4, true>), dim3(ff1_grid(nblk)), dim3(G_THREADS), 0, st, p);
    }
    return check_launch("ff1_bf16_mfma_kernel");
}

}  // namespace griffin
