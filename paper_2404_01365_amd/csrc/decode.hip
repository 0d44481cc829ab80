// Generation phase: one token through a (compact or full) gated FF block
// (Section 4.2 "Generation with Expert Neurons"; Eq. 1 and Eq. 4-5):
//     z_j = sigma(wg_j . x + bg_j) * (w1_j . x + b1_j),   y = sum_j z_j W2[j][:] + b2.
//
// One pass over 3*n*d weights at one flop per byte: the kernel is shaped by what HBM likes.
// Measured on MI355X, read bandwidth is highest when the requests in flight at any moment
// cover a compact window of addresses and each CU keeps only ~32-64 KB outstanding; many
// lightly loaded waves beat few waves with deep queues.  So:
//   * a TEAM of R wavefronts owns a neuron: wave r streams the r-th 1 KB piece of the
//     neuron's three rows (16 bytes per lane), so a wave holds only its slab of x (one chunk)
//     and of y (one chunk of fp32 accumulators) and registers do not limit occupancy;
//   * teams take neurons round-robin across the whole chip (team T, step s -> neurons
//     (s*NT + T)*G ... +G-1), so at any time the chip reads one contiguous window of rows
//     per matrix (one window in all when the three rows of a neuron are stored side by
//     side, i.e. Wg, W1, W2 interleaved with ld = 3d);
//   * the dot products (two per row of x) are reduced inside the wave with DPP, those of several rows together, combined
//     across the team's waves through a few LDS words and one barrier per G neurons, and the loads of the next
//     two steps are already in flight while that happens (three register sets; the loads are
//     branch-free so the compiler waits for the oldest set only; with one step of lookahead a
//     wave streams only one step's bytes per memory latency, which is what bounds narrow rows);
//   * each workgroup folds its teams' y slabs in LDS (one team for rows of 4 KB and more) and
//     writes one fp32 partial row; a second tiny kernel adds the partial rows in a fixed
//     order (deterministic), adds b2 and converts to the output type.
#include "common.h"

namespace griffin {

constexpr int DEC_G = 1;                 // neurons per team step
constexpr int DEC_MAX_WAVES = 16;        // waves per workgroup
constexpr int DEC_MAX_TEAMS = 8;         // teams per workgroup
constexpr int DEC_MAX_PARTS = 256;       // partial rows per batch row
constexpr int DEC_NB_MAX = 4;            // rows of x sharing one pass over the weights
constexpr int DEC_MAX_D = 8192;
// LDS floats for folding teams: a workgroup has several only where a team has four waves at the most.  (Room for all 8192 columns
// beside the partial sums of four rows makes 64 KB, two workgroups a CU where there were three: 25 fp32 rows of 120 x 191
// 17.6 us a call against 14.1.)
constexpr int DEC_FOLD_FLOATS = 4 * 64 * 8;

// partial sums per value and team: one per wave where each value is summed over its wave, four where NB rows go together
constexpr int dec_red_width(int NB) { return NB == 1 ? 16 : 64; }

struct DecodeParams {
    const void *Wg, *W1, *W2, *bg, *b1;
    const int32_t *idx;
    const void *x;
    float *part;
    int64_t ld;
    int32_t d, n, n_src, act, P, batch;
    int32_t R, teams;        // waves per team, teams per workgroup
};

struct MultiPtrs {
    const void *p[GRIFFIN_MAX_BATCH][5];   // Wg, W1, W2, bg, b1 of every row's own block
};

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
// cache-policy bits of a raw buffer store on gfx942/gfx950: sc0 (bit 0) and sc1 (bit 4) = write through to memory
[[maybe_unused]] constexpr int DEC_AUX_WRITE_THROUGH = 1 | 16;

// by value on purpose: bit-casting a vector element expression (v.y) in place picks element 0
__device__ __forceinline__ bf16x2 as_bf16x2(uint32_t v) { return __builtin_bit_cast(bf16x2, v); }

// A 16-byte chunk of a row: 8 bf16 or 4 fp32 elements.
template <bool BF16>
struct Chunk {
    static constexpr int E = BF16 ? 8 : 4;
    static __device__ __forceinline__ float dot(const u32x4 &w, const u32x4 &x)
    {
        float acc = 0.0f;
        if (BF16) {
            acc = __builtin_amdgcn_fdot2_f32_bf16(as_bf16x2(w.x), as_bf16x2(x.x), acc, false);
            acc = __builtin_amdgcn_fdot2_f32_bf16(as_bf16x2(w.y), as_bf16x2(x.y), acc, false);
            acc = __builtin_amdgcn_fdot2_f32_bf16(as_bf16x2(w.z), as_bf16x2(x.z), acc, false);
            acc = __builtin_amdgcn_fdot2_f32_bf16(as_bf16x2(w.w), as_bf16x2(x.w), acc, false);
        } else {
            acc = fmaf(__uint_as_float(w.x), __uint_as_float(x.x), acc);
            acc = fmaf(__uint_as_float(w.y), __uint_as_float(x.y), acc);
            acc = fmaf(__uint_as_float(w.z), __uint_as_float(x.z), acc);
            acc = fmaf(__uint_as_float(w.w), __uint_as_float(x.w), acc);
        }
        return acc;
    }
    static __device__ __forceinline__ void axpy(float z, const u32x4 &w, float (&y)[8])
    {
        if (BF16) {
            y[0] = fmaf(z, bf16_lo(w.x), y[0]); y[1] = fmaf(z, bf16_hi(w.x), y[1]);
            y[2] = fmaf(z, bf16_lo(w.y), y[2]); y[3] = fmaf(z, bf16_hi(w.y), y[3]);
            y[4] = fmaf(z, bf16_lo(w.z), y[4]); y[5] = fmaf(z, bf16_hi(w.z), y[5]);
            y[6] = fmaf(z, bf16_lo(w.w), y[6]); y[7] = fmaf(z, bf16_hi(w.w), y[7]);
        } else {
            y[0] = fmaf(z, __uint_as_float(w.x), y[0]); y[1] = fmaf(z, __uint_as_float(w.y), y[1]);
            y[2] = fmaf(z, __uint_as_float(w.z), y[2]); y[3] = fmaf(z, __uint_as_float(w.w), y[3]);
        }
    }
};

// Passes of two to four rows.  The sums of NV values (2, 4 or 8) over the sixteen lanes of every DPP row, value i in the lanes
// whose index ends in i (log2 NV bits).  Two values that are added over the same pair of lanes change places while they are
// added, so a step halves the number of values: 22 instructions for eight values, where a sum of each over the wavefront takes 88
// (which bound the passes of three and four rows: three rows of 4096 x 5504 36.8 -> 29.1 us, of 3072 x 12288 68 -> 44, of a
// 4096 x 11008 Eq. 2 block 51.4 -> 37.8).  A row that goes alone has one or two values and waits for memory; it keeps the plain sum,
// because the exchange takes its registers across a step of occupancy and a launch of 256 workgroups per row needs three of
// them on a CU (three own-set rows, k = n/2, of 4096 x 14336 98 us with it and 88 without, of 2752 x 8000 49.8 and 37.7).
template <int CTRL>
__device__ __forceinline__ float pair_step(float even, float odd, bool is_odd)
{
    return (is_odd ? odd : even) + dpp_f32<CTRL>(is_odd ? even : odd);
}

template <int NV>
__device__ __forceinline__ float row16_sums(const float (&v)[NV], int lane)
{
    constexpr int XOR1 = 0xB1, XOR2 = 0x4E, ROR4 = 0x124, ROR8 = 0x128;
    const bool o0 = lane & 1, o1 = lane & 2, o2 = lane & 4;
    float a[4], b[2], c;
#pragma unroll
    for (int i = 0; i < NV / 2; ++i)
        a[i] = pair_step<XOR1>(v[2 * i], v[2 * i + 1], o0);
    if (NV >= 4) {
#pragma unroll
        for (int i = 0; i < NV / 4; ++i)
            b[i] = pair_step<XOR2>(a[(2 * i) % 4], a[(2 * i + 1) % 4], o1);
    } else {
        b[0] = a[0] + dpp_f32<XOR2>(a[0]);
    }
    // a rotation by four brings a lane whose bit 2 differs and whose lower bits agree
    c = NV >= 8 ? pair_step<ROR4>(b[0], b[1], o2) : b[0] + dpp_f32<ROR4>(b[0]);
    return c + dpp_f32<ROR8>(c);
}

// z of the team's neuron for NB rows from the partial sums [value][4 per wave, zero up to 64] (value: gate and up of row 0, of
// row 1, ...).  The lanes share the values out, 64 / NV lanes each; sigma is taken once for all rows where a row's gate and
// up sums are in one DPP row.
template <bool GATED, int NB>
__device__ __forceinline__ void team_z(const float (*red)[64], int lane, int act, float bg, float b1, float (&z)[NB])
{
    constexpr int NV = (GATED ? 2 : 1) * NB, LPV = 64 / NV;
    const float *src = &red[lane / LPV][(lane % LPV) * NV];
    float q = 0.0f;
    if (NV == 8) {
        const f32x4 t = *(const f32x4 *)src, u = *(const f32x4 *)(src + 4);
        q = ((t.x + t.y) + (t.z + t.w)) + ((u.x + u.y) + (u.z + u.w));
    } else if (NV == 4) {
        const f32x4 t = *(const f32x4 *)src;
        q = (t.x + t.y) + (t.z + t.w);
    } else {
        const float2 t = *(const float2 *)src;
        q = t.x + t.y;
    }
    q += dpp_f32<0xB1>(q);
    q += dpp_f32<0x4E>(q);
    q += dpp_f32<0x141>(q);          // eight lanes
    if (NV == 8) {
        // row nb: gate in its lanes 0-7, up in its lanes 8-15
        const float u = dpp_f32<0x128>(q);
        const float zl = act_apply(act, q + bg) * (u + b1);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            z[nb] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(zl), 16 * nb));
        return;
    }
    q += dpp_f32<0x140>(q);          // sixteen
#define TEAM_ROW(r_) __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q), 16 * (r_)))
    if (NV == 4 && !GATED) {
        const float zl = act_apply(act, q + b1);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            z[nb] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(zl), 16 * nb));
    } else if (NV == 4) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            z[nb] = act_apply(act, TEAM_ROW(2 * nb) + bg) * (TEAM_ROW(2 * nb + 1) + b1);
    } else {                         // two rows of an Eq. 2 block
        z[0] = act_apply(act, TEAM_ROW(0) + TEAM_ROW(1) + b1);
        z[NB - 1] = act_apply(act, TEAM_ROW(2) + TEAM_ROW(3) + b1);
    }
#undef TEAM_ROW
}

// GATED and INDEXED are compile-time so that the three row loads of a neuron are issued
// back to back with no branch between them (a branch there makes the compiler wait for the
// first load before issuing the next).
// NB = rows of x that share the block's weights in one pass (the weights are streamed once for
// NB rows; 1 for the per-row variants).
template <bool BF16, bool GATED, bool INDEXED, bool BIAS, int NB>
__device__ __forceinline__ void decode_body(const DecodeParams &p, const void *Wg, const void *W1,
                                            const void *W2, const void *bg, const void *b1,
                                            float (*red)[2 * NB][dec_red_width(NB)], float *fold)
{
    constexpr int E = Chunk<BF16>::E;
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int G = DEC_G, NMAT = GATED ? 2 : 1;
    static_assert(G == 1, "the team's sums are those of one neuron");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, in an SGPR
    const int R = p.R;
    const int team = wave / R, wt = wave - team * R;
    const int b = blockIdx.y * NB;           // first of this block's NB rows
    const int d = p.d, nch = d / E;

    const int c = wt * 64 + lane;            // this lane's 16-byte chunk of every row
    const bool valid = c < nch;
    const int cc = valid ? c : nch - 1;      // clamped: loads stay in bounds, x = 0 kills the terms
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    u32x4 xr[NB];
    float ya[NB][8];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const bool live = valid && b + nb < p.batch;     // rows past the batch behave as x = 0
        xr[nb] = live ? ((const u32x4 *)((const char *)p.x + (int64_t)(b + nb) * d * ES))[cc] : zero4;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            ya[nb][e] = 0.0f;
    }

    const int NT = gridDim.x * p.teams;              // teams on the chip for this batch row
    const int T = blockIdx.x * p.teams + team;
    const int nsteps = (p.n + NT * G - 1) / (NT * G);
    const int32_t *idx = INDEXED ? p.idx + (int64_t)b * p.n : nullptr;
    const int64_t row_bytes = p.ld * ES;
    constexpr int NV = NMAT * NB;                    // values to combine across the team per step
    constexpr int RW = dec_red_width(NB);
    float(*myred)[2 * NB][RW] = red + team * 2;       // [parity][value][partial sums of the team's waves]


    // Loads are branch-free (slots past the last neuron re-read the last row, which stays in
    // L2, and are masked when z is formed) so that the compiler can wait for exactly the
    // older buffer while the newer one is still in flight.
    u32x4 buf[3][G][3];
    int rows[3][G];
    float bias[3][G][2];
    // a bias that is not there is loaded from a matrix instead (at an element that exists) and not used: a branch around its load
    // would make it, and the weights behind it, wait (4096 x 11008 Eq. 2 with biases, 3 rows: 45.0 us a call against 38.2)
    const void *bgp = bg ? bg : W1, *b1p = b1 ? b1 : W1;

// the weights are read once per call: non-temporal loads (no allocation in the caches on the way)
// stream measurably faster than plain ones (135 MB: 20.4 us against 24.0 us in a bare read loop)
#define DEC_STREAM_LOAD(ptr_) __builtin_nontemporal_load(ptr_)
#define DEC_LOAD(B_, s_)                                                                     \
    {                                                                                        \
        _Pragma("unroll") for (int g = 0; g < G; ++g)                                        \
        {                                                                                    \
            const int j_ = min(((s_) * NT + T) * G + g, p.n - 1);                            \
            int row_ = j_;                                                                   \
            if (INDEXED) {                                                                   \
                row_ = idx[j_];                                                              \
                row_ = row_ < 0 ? 0 : (row_ >= p.n_src ? p.n_src - 1 : row_);                \
            }                                                                                \
            if (GATED)                                                                       \
                buf[B_][g][0] = DEC_STREAM_LOAD((const u32x4 *)((const char *)Wg + row_ * row_bytes) + cc); \
            buf[B_][g][1] = DEC_STREAM_LOAD((const u32x4 *)((const char *)W1 + row_ * row_bytes) + cc);     \
            buf[B_][g][2] = DEC_STREAM_LOAD((const u32x4 *)((const char *)W2 + row_ * row_bytes) + cc);     \
            if (BIAS) {                                                                      \
                if (GATED)                                                                   \
                    bias[B_][g][0] = load_scalar<BF16>(bgp, row_);                           \
                bias[B_][g][1] = load_scalar<BF16>(b1p, row_);                               \
            }                                                                                \
            rows[B_][g] = row_;                                                              \
        }                                                                                    \
    }

#define DEC_CONSUME(B_, s_)                                                                  \
    {                                                                                        \
        float pv_[NV];                                                                       \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                    \
        {                                                                                    \
            if (GATED)                                                                       \
                pv_[nb * NMAT] = Chunk<BF16>::dot(buf[B_][0][0], xr[nb]);                    \
            pv_[nb * NMAT + NMAT - 1] = Chunk<BF16>::dot(buf[B_][0][1], xr[nb]);             \
        }                                                                                    \
        const float bg_ = BIAS && GATED && bg ? bias[B_][0][0] : 0.0f, b1_ = BIAS && b1 ? bias[B_][0][1] : 0.0f; \
        float z_[NB];                                                                        \
        if constexpr (NB == 1) {                                                             \
            _Pragma("unroll") for (int v = 0; v < NV; ++v) pv_[v] = wave_sum(pv_[v]);        \
            if (lane == 0) {                                                                 \
                _Pragma("unroll") for (int v = 0; v < NV; ++v) myred[(s_) & 1][v][wt] = pv_[v]; \
            }                                                                                \
            __syncthreads();                                                                 \
            const float q_ = row16_sum((lane >> 4) < NV ? myred[(s_) & 1][lane >> 4][lane & 15] : 0.0f); \
            const float g_ = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q_), 0)); \
            const float u_ = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q_), 16 * (NV - 1))); \
            z_[0] = GATED ? act_apply(p.act, g_ + bg_) * (u_ + b1_) : act_apply(p.act, u_ + b1_); \
        } else {                                                                             \
            const float part_ = row16_sums<NV>(pv_, lane);                                   \
            if ((lane & 15) < NV)                                                            \
                myred[(s_) & 1][lane & 15][wt * 4 + (lane >> 4)] = part_;                    \
            __syncthreads();                                                                 \
            team_z<GATED, NB>(myred[(s_) & 1], lane, p.act, bg_, b1_, z_);                   \
        }                                                                                    \
        const int j_ = (s_) * NT + T;                                                        \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                    \
            Chunk<BF16>::axpy(j_ < p.n ? z_[nb] : 0.0f, buf[B_][0][2], ya[nb]);              \
    }

    if (nsteps > 0) {
        DEC_LOAD(0, 0)
        DEC_LOAD(1, 1)             // steps past the end re-read the last row and contribute nothing
    }
    // zero the padding entries of the cross-wave buffers once (the first rows are already on their way)
    constexpr int RQ = RW / 4;
    for (int i = threadIdx.x; i < p.teams * 2 * NV * RQ; i += blockDim.x)
        *(f32x4 *)&red[i / (NV * RQ)][(i / RQ) % NV][i % RQ * 4] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
    __syncthreads();
    for (int s = 0; s < nsteps; s += 3) {
        DEC_LOAD(2, s + 2)
        DEC_CONSUME(0, s)
        if (s + 1 >= nsteps)
            break;
        DEC_LOAD(0, s + 3)
        DEC_CONSUME(1, s + 1)
        if (s + 2 >= nsteps)
            break;
        DEC_LOAD(1, s + 4)
        DEC_CONSUME(2, s + 2)
    }
#undef DEC_LOAD
#undef DEC_STREAM_LOAD
#undef DEC_CONSUME
    (void)rows;

    // fold the workgroup's teams (fixed order), then one fp32 partial row per workgroup and x row
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        for (int t = 1; t < p.teams; ++t) {
            if (team == t && valid) {
#pragma unroll
                for (int e = 0; e < E; e += 4)
                    *(float4 *)(fold + c * E + e) = make_float4(ya[nb][e], ya[nb][e + 1], ya[nb][e + 2], ya[nb][e + 3]);
            }
            __syncthreads();
            if (team == 0 && valid) {
#pragma unroll
                for (int e = 0; e < E; e += 4) {
                    const float4 v = *(const float4 *)(fold + c * E + e);
                    ya[nb][e] += v.x; ya[nb][e + 1] += v.y; ya[nb][e + 2] += v.z; ya[nb][e + 3] += v.w;
                }
            }
            __syncthreads();
        }
        // The partial row is private to this kernel and the one that adds the rows up, so its columns are
        // stored in the order that makes every store instruction one contiguous kilobyte: quad e/4 of
        // chunk c goes to float4 slot (e/4) * nch + c (a lane's 8 columns would otherwise leave as two
        // instructions that each fill every other 16 bytes).  The stores are write-through (sc0 sc1): the rows
        // then sit in memory when the kernel ends instead of as dirty lines in eight L2s that the end of the
        // kernel has to write back before the adding kernel may start (0.4 us per layer-token less than with
        // plain or non-temporal stores, measured on three shapes).
        if (team == 0 && valid && b + nb < p.batch) {
#if defined(__HIP_DEVICE_COMPILE__)      // the host pass has no buffer builtins
            float *out = p.part + ((int64_t)(b + nb) * p.P + blockIdx.x) * d;
            const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void *)out, 0, 0x7FFFFFFE, 0x00020000);
#pragma unroll
            for (int e = 0; e < E; e += 4) {
                const f32x4 v = {ya[nb][e], ya[nb][e + 1], ya[nb][e + 2], ya[nb][e + 3]};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rp, ((e / 4) * nch + c) * 16, 0,
                                                       DEC_AUX_WRITE_THROUGH);
            }
#endif
        }
    }
}

template <bool BF16, bool GATED, bool INDEXED, bool BIAS, int NB>
__global__ __launch_bounds__(DEC_MAX_WAVES * 64) void ff_decode_kernel(DecodeParams p)
{
    __shared__ __attribute__((aligned(16))) float red[DEC_MAX_TEAMS * 2][2 * NB][dec_red_width(NB)];
    __shared__ __attribute__((aligned(16))) float fold[DEC_FOLD_FLOATS];
    decode_body<BF16, GATED, INDEXED, BIAS, NB>(p, p.Wg, p.W1, p.W2, p.bg, p.b1, red, fold);
}

template <bool BF16, bool GATED, bool BIAS>
__global__ __launch_bounds__(DEC_MAX_WAVES * 64) void ff_decode_multi_kernel(DecodeParams p, MultiPtrs m)
{
    __shared__ __attribute__((aligned(16))) float red[DEC_MAX_TEAMS * 2][2][dec_red_width(1)];
    __shared__ __attribute__((aligned(16))) float fold[DEC_FOLD_FLOATS];
    const void *const *q = m.p[blockIdx.y];
    decode_body<BF16, GATED, false, BIAS, 1>(p, q[0], q[1], q[2], q[3], q[4], red, fold);
}

struct B2Ptrs {
    const void *p[GRIFFIN_MAX_BATCH];    // b2 of every row's own block (multi path)
};

// y[b] = sum_p part[b][p] + b2, the rows p taken in a fixed order.  A workgroup of eight wavefronts owns
// RED_Q float4 slots (one 128-byte line) of every partial row: lane (r, q) of wave w reads slot q of the
// rows p = 8 w + r, + 64, + 128, + 192 (all four loads on their way at once; a wave instruction covers
// eight whole lines), adds them in that order, the eight lanes of a slot are added with wave shuffles and
// the eight waves through LDS.  nch > 0 says that the rows come from the streaming kernel, which stores
// quad h of 16-byte chunk c at slot h * nch + c (bf16 blocks: 8 columns per chunk); 0 = columns in order.
constexpr int RED_Q = 8, RED_WAVES = 8;
template <bool BF16, bool MULTI>
__global__ __launch_bounds__(RED_WAVES * 64) void ff_decode_reduce_kernel(const float *part, int P, int d, int nch,
                                                                           const void *b2_one, B2Ptrs b2_multi,
                                                                           void *y)
{
    __shared__ float4 fold[RED_WAVES][RED_Q];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b = blockIdx.y;
    const int r = lane >> 3, qi = lane & 7;
    const int nq = d >> 2;
    const int q = blockIdx.x * RED_Q + qi;
    const int qc = q < nq ? q : nq - 1;            // clamped: loads stay in bounds, the result is not stored
    const float *base = part + (int64_t)b * P * d + (int64_t)qc * 4;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int p0 = wave * 8 + r; p0 < P; p0 += 256) {
        float4 t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int pp = p0 + 64 * i;
            const f32x4 v = pp < P ? __builtin_nontemporal_load((const f32x4 *)(base + (int64_t)pp * d)) : (f32x4){0.f, 0.f, 0.f, 0.f};
            t[i] = make_float4(v.x, v.y, v.z, v.w);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc.x += t[i].x; acc.y += t[i].y; acc.z += t[i].z; acc.w += t[i].w;
        }
    }
    // the eight lanes (r = 0..7) that hold the same slot
#pragma unroll
    for (int m = 8; m < 64; m <<= 1) {
        acc.x += __shfl_xor(acc.x, m, 64); acc.y += __shfl_xor(acc.y, m, 64);
        acc.z += __shfl_xor(acc.z, m, 64); acc.w += __shfl_xor(acc.w, m, 64);
    }
    if (r == 0)
        fold[wave][qi] = acc;
    __syncthreads();
    if (threadIdx.x < RED_Q && q < nq) {
        float4 s = fold[0][qi];
#pragma unroll
        for (int w = 1; w < RED_WAVES; ++w) {
            const float4 v = fold[w][qi];
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        const int c = nch > 0 ? (q % nch) * 8 + (q / nch) * 4 : q * 4;      // first of this slot's four columns
        const void *b2 = MULTI ? b2_multi.p[b] : b2_one;
        if (b2) {
            s.x += load_scalar<BF16>(b2, c);
            s.y += load_scalar<BF16>(b2, c + 1);
            s.z += load_scalar<BF16>(b2, c + 2);
            s.w += load_scalar<BF16>(b2, c + 3);
        }
        const int64_t o = (int64_t)b * d + c;
        if (BF16) {
            uint2 w;
            w.x = f32x2_to_bf16x2(s.x, s.y);
            w.y = f32x2_to_bf16x2(s.z, s.w);
            *(uint2 *)((uint16_t *)y + o) = w;
        } else {
            *(float4 *)((float *)y + o) = s;
        }
    }
}

// grid of the kernel above for rows of d floats
static dim3 reduce_grid(int d, int batch) { return dim3((d / 4 + RED_Q - 1) / RED_Q, batch); }

// waves per team for a row of d elements, 0 if this build cannot cover it
static int decode_team_waves(int32_t d, bool bf16)
{
    const int nch = d / (bf16 ? 8 : 4);
    const int R = (nch + 63) / 64;
    return (R <= DEC_MAX_WAVES && d <= DEC_MAX_D) ? R : 0;
}

// workgroups (= partial rows) per batch row: enough to fill the chip when the rows of a batch
// are taken DEC_NB_MAX at a time
int decode_parts(int32_t n, int32_t batch)
{
    const int groups = batch <= 2 ? 1 : (batch + DEC_NB_MAX - 1) / DEC_NB_MAX;
    int P = (512 + groups - 1) / groups;
    if (P > DEC_MAX_PARTS) P = DEC_MAX_PARTS;
    if (P < 8) P = 8;
    const int by_work = (n + 2 * DEC_G - 1) / (2 * DEC_G);
    if (P > by_work) P = by_work;
    // A multiple of the eight XCDs: else the slices of the grid start on different ones and some get more workgroups than they
    // hold at once (12 rows of 320 x 1000 with P = 170 19.3 us, 168 13.9; 18 fp32 rows of 192 x 250 with 102 18.3, 96 13.9)
    if (P >= 16) P &= ~7;
    return P < 1 ? 1 : P;
}

// What a decode has to be given: a partial row per workgroup and batch row; for the shapes whose batches have always run
// on the matrix cores also what sixteen rows a pass need there (partial rows, Z and membership words).
size_t decode_least_floats(int32_t d, int32_t n, int32_t batch)
{
    size_t floats = (size_t)decode_parts(n, batch) * batch * d;
    if (decode_whole_pieces(d, batch) && n >= 64 && n <= 32768) {
        int64_t nr = 256 / (d / 512);
        if (nr > 64) nr = 64;
        if (nr < (n + 479) / 480) nr = (n + 479) / 480;
        const size_t fb = (size_t)batch * nr * d + (size_t)n * 17 + 128;
        if (fb > floats)
            floats = fb;
    }
    return floats;
}

// What it makes use of: more rows a pass want more room for their Z, and the matrix-core path also takes shapes that
// it did not take before.  A decode that fits the library's own array goes on fitting it: the two entry points choose
// their route by the shape alone.
static size_t decode_route_floats(int32_t d, int32_t n, int32_t batch)
{
    const size_t least = decode_least_floats(d, n, batch), own = DEC_STATIC_BYTES / sizeof(float);
    return batch < DEC_MASKED_MIN_ROWS ? 0 : decode_batch_floats(d, n, batch, least <= own ? own : (size_t)-1);
}

size_t decode_wanted_floats(int32_t d, int32_t n, int32_t batch)
{
    const size_t least = decode_least_floats(d, n, batch), route = decode_route_floats(d, n, batch);
    return route > least ? route : least;
}

// one-shot instrumentation: events recorded around the streaming kernel of the next decode
static thread_local hipEvent_t g_probe_begin = nullptr, g_probe_mid = nullptr, g_probe_end = nullptr;

void set_decode_probe(hipEvent_t begin, hipEvent_t mid, hipEvent_t end)
{
    g_probe_begin = begin;
    g_probe_mid = mid;
    g_probe_end = end;
}

// Bytes that the matrix-core path has to spare against rows that go four at a time through a shared block, or one by one through
// their own sets: it has three kernels instead of two, partial rows of its own (600 bytes per row and column pay for them) and,
// for own sets, the membership words to form; groups of four run side by side and share what the caches hold, passes do not.
//   * own sets, one by one / masked, us: 704 x 4000, k = n/2: 5 rows 15.8 / 22.1 (25 MB spared), 8 rows 22.7 / 23.0 (51), k = 3n/4:
//     27.5 / 22.6 (84); 40 rows of 1408 x 5632, k = n/20 29.7 / 39.7 (47), k = n/10 43.8 / 39.3 (142); 5 rows of 2752 x 15520, k = n/3
//     80 / 60 (167); three and four rows: 100 MB.  4 rows of 4096 x 14336, k = n/3 90 / 72 (141), k = n/2 120 / 72 (352); 3 rows of
//     2752 x 15520, k = n/2 62 / 63 (110), 4 rows of 5632 x 12428, k = n/3 101 / 101 (168);
//   * a shared Eq. 3 block, four at a time / matrix cores, us: 704 wide, 8 rows n = 12784 25.5 / 25.6 (54), 12 rows n = 6392
//     21.1 / 19.9 (54), 16 rows n = 2982 16.5 / 16.5 (38), 33 rows n = 2130 20.7 / 21.5 (72); 4288 wide, 8 rows n = 349 22.0 / 21.6 (9),
//     16 rows n = 489 26.2 / 25.1 (38), 33 rows (two passes) n = 1049 51.5 / 54.3 (189); 5632 wide, 17 rows (two passes) n = 2308
//     62.8 / 63.4 (234), 33 rows (three) 95.0 / 97.1 (468).
static int64_t dec_batch_spare(int32_t d, int32_t batch, int passes, bool own_sets)
{
    const int64_t partials = (int64_t)600 * batch * d;
    if (own_sets)
        return batch < DEC_BATCH_MIN_ROWS ? 100000000 : 40000000 + partials;
    return (d <= 2800 ? 50000000 : 16000000) + (batch > 16 ? partials : 0) + (int64_t)100000000 * (passes - 1);
}

int launch_decode(const DecodeJob &job, hipStream_t st)
{
    const int R = decode_team_waves(job.d, job.bf16);
    if (R == 0)
        return GRIFFIN_EUNSUPPORTED;
    int P = decode_parts(job.n, job.batch);
    // A batch through one shared block takes the matrix-core path, with as many rows a pass as the workspace has room
    // for; else rows go four at a time.  A batch whose rows have their own sets inside one block takes it as a masked pass
    // over the whole block if the workspace was sized for the whole block; else rows go one by one through the index lists.
    // Rows of other widths than whole 1 KB pieces up to 5120 take it when the bytes it spares pay for it (dec_batch_spare).
    const int32_t nb = job.idx ? job.n_src : job.n;
    size_t have = 0;
    if (job.bf16 && !job.multi && job.W2 && job.batch >= (job.idx ? DEC_MASKED_MIN_ROWS : DEC_BATCH_MIN_ROWS)) {
        have = decode_route_floats(job.d, nb, job.batch);
        // own sets: a workspace sized for the whole block; where these batches have always run here, also the size that has always
        // done, as long as it is not what a workspace for k neurons has
        if (job.idx && job.part_bytes < decode_wanted_floats(job.d, nb, job.batch) * sizeof(float)) {
            const bool least = decode_whole_pieces(job.d, job.batch) && job.part_bytes >= decode_least_floats(job.d, nb, job.batch) * sizeof(float);
            if (!least || (job.n < nb && job.part_bytes <= decode_wanted_floats(job.d, job.n, job.batch) * sizeof(float)))
                have = 0;
        }
        if (have > job.part_bytes / sizeof(float))
            have = job.part_bytes / sizeof(float);
        const int passes = decode_batch_passes(job.d, nb, job.batch, have);
        const int64_t rows_read = job.idx ? (int64_t)job.batch * job.n : (int64_t)((job.batch + DEC_NB_MAX - 1) / DEC_NB_MAX) * nb;
        const int64_t spared = (rows_read - (int64_t)passes * nb) * (job.Wg ? 6 : 4) * job.d;
        if (passes == 0 || !(decode_whole_pieces(job.d, job.batch) || spared > dec_batch_spare(job.d, job.batch, passes, job.idx != nullptr)))
            have = 0;
    }
    const bool batch_path = have > 0;
    if (!batch_path && job.part_bytes < (size_t)P * job.batch * job.d * sizeof(float))
        return GRIFFIN_EWORKSPACE;

    DecodeParams p;
    p.Wg = job.Wg; p.W1 = job.W1; p.W2 = job.W2; p.bg = job.bg; p.b1 = job.b1;
    p.idx = job.idx; p.n_src = job.idx ? job.n_src : job.n;
    p.x = job.x; p.part = job.part; p.ld = job.ld;
    p.d = job.d; p.n = job.n; p.act = job.act; p.P = P; p.batch = job.batch;
    p.R = R;
    // about eight waves per workgroup, one workgroup per CU: measured best (more waves or
    // more loads in flight per CU lower the achieved bandwidth)
    p.teams = R >= 8 ? 1 : 8 / R;

    MultiPtrs m;
    B2Ptrs b2m;
    for (int b = 0; b < GRIFFIN_MAX_BATCH; ++b)
        b2m.p[b] = nullptr;
    const void *b2 = job.b2;
    if (job.multi) {
        for (int b = 0; b < job.batch; ++b) {
            const griffin_layer &c = job.multi[b];
            m.p[b][0] = c.Wg; m.p[b][1] = c.W1; m.p[b][2] = c.W2; m.p[b][3] = c.bg; m.p[b][4] = c.b1;
            b2m.p[b] = c.b2;
        }
        for (int b = job.batch; b < GRIFFIN_MAX_BATCH; ++b)
            for (int q = 0; q < 5; ++q)
                m.p[b][q] = nullptr;
    }

    const hipEvent_t ev_begin = g_probe_begin, ev_mid = g_probe_mid, ev_end = g_probe_end;
    g_probe_begin = g_probe_mid = g_probe_end = nullptr;
    if (ev_begin && hipEventRecord(ev_begin, st) != hipSuccess)
        return set_hip_error(hipGetLastError(), "hipEventRecord");

    if (decode_split_supported(job)) {
        int rc = launch_decode_split(job, st, ev_mid);
        if (rc == GRIFFIN_OK && ev_end && hipEventRecord(ev_end, st) != hipSuccess)
            return set_hip_error(hipGetLastError(), "hipEventRecord");
        return rc;
    }
    if (!job.W2 && !job.multi)
        return GRIFFIN_EUNSUPPORTED;       // only the transposed copy is there and this call cannot use it
    if (batch_path) {
        // the caller's words are read where griffin.h says so; for other shapes they need not have been built
        const uint32_t *sets = decode_whole_pieces(job.d, job.batch) ? job.sets : nullptr;
        int rc = job.idx ? launch_decode_batch_front(job, job.n_src, job.idx, job.n, sets, have, &P, st)
                         : launch_decode_batch_front(job, job.n, nullptr, 0, nullptr, have, &P, st);
        if (rc != GRIFFIN_OK)
            return rc;
        if (ev_mid && hipEventRecord(ev_mid, st) != hipSuccess)
            return set_hip_error(hipGetLastError(), "hipEventRecord");
        dim3 rgrid = reduce_grid(job.d, job.batch), rblock(RED_WAVES * 64);
        hipLaunchKernelGGL((ff_decode_reduce_kernel<true, false>), rgrid, rblock, 0, st, job.part, P, job.d, 0, b2, b2m, job.y);
        rc = check_launch("ff_decode_reduce_kernel");
        if (rc == GRIFFIN_OK && ev_end && hipEventRecord(ev_end, st) != hipSuccess)
            return set_hip_error(hipGetLastError(), "hipEventRecord");
        return rc;
    }

    // rows through one shared block are taken NB at a time (weights streamed once per NB rows)
    const bool shared_block = !job.multi && !job.idx;
    const int NB = !shared_block || job.batch == 1 ? 1 : (job.batch == 2 ? 2 : DEC_NB_MAX);
    dim3 grid(P, (job.batch + NB - 1) / NB), block(p.teams * R * 64);
    const bool gated = job.multi ? job.multi[0].Wg != nullptr : job.Wg != nullptr;
    const bool indexed = job.idx != nullptr;
    const bool bias = job.multi ? (job.multi[0].bg || job.multi[0].b1) : (job.bg || job.b1);
#define DEC_GO1(BF, GA, IX, BI, NB_) hipLaunchKernelGGL((ff_decode_kernel<BF, GA, IX, BI, NB_>), grid, block, 0, st, p)
#define DEC_GO(BF, GA, IX, BI)                                         \
    {                                                                  \
        if (IX || NB == 1) DEC_GO1(BF, GA, IX, BI, 1);                 \
        else if (NB == 2) DEC_GO1(BF, GA, false, BI, 2);               \
        else DEC_GO1(BF, GA, false, BI, DEC_NB_MAX);                   \
    }
    // Per-row blocks of more than eight waves a team: one workgroup a CU, by asking for more than half of its LDS.  Two of ten waves
    // each, at the registers of these kernels, stream 10 % slower (5120 x 6912 Eq. 3, 4 / 8 rows: with biases 152 / 301 us against
    // 136 / 277, without 151 / 295 against 138 / 276; Eq. 2 98 / 204 against 95 / 186; 6144 x 5500 135 / 270 against 130 / 260; 8192
    // wide, where two do not fit, the same; up to 4096 wide two and three are the better number).
    const int alone = R > 8 ? 72 * 1024 : 0;
#define DEC_GO_MULTI(BF, GA, BI)                                                                                   \
    {                                                                                                              \
        if (alone)                                                                                                 \
            RAISE_LDS_LIMIT((ff_decode_multi_kernel<BF, GA, BI>), alone)                                           \
        hipLaunchKernelGGL((ff_decode_multi_kernel<BF, GA, BI>), grid, block, alone, st, p, m);                    \
    }
#define DEC_PICK3(BF, GA, IX) { if (bias) DEC_GO(BF, GA, IX, true) else DEC_GO(BF, GA, IX, false) }
#define DEC_PICK2(BF, GA) { if (indexed) DEC_PICK3(BF, GA, true) else DEC_PICK3(BF, GA, false) }
#define DEC_PICKM(BF, GA) { if (bias) DEC_GO_MULTI(BF, GA, true) else DEC_GO_MULTI(BF, GA, false) }
    if (job.multi) {
        if (job.bf16) { if (gated) DEC_PICKM(true, true) else DEC_PICKM(true, false) }
        else          { if (gated) DEC_PICKM(false, true) else DEC_PICKM(false, false) }
    } else if (job.bf16) {
        if (gated) DEC_PICK2(true, true) else DEC_PICK2(true, false)
    } else {
        if (gated) DEC_PICK2(false, true) else DEC_PICK2(false, false)
    }
#undef DEC_PICK3
#undef DEC_PICK2
#undef DEC_PICKM
#undef DEC_GO
#undef DEC_GO1
#undef DEC_GO_MULTI
    int rc = check_launch("ff_decode_kernel");
    if (rc != GRIFFIN_OK)
        return rc;
    if (ev_mid && hipEventRecord(ev_mid, st) != hipSuccess)
        return set_hip_error(hipGetLastError(), "hipEventRecord");

    dim3 rgrid = reduce_grid(job.d, job.batch), rblock(RED_WAVES * 64);
    const int nch = job.bf16 ? job.d / 8 : 0;       // the streaming kernel's order of columns (fp32 rows: in order)
    if (job.multi) {
        if (job.bf16)
            hipLaunchKernelGGL((ff_decode_reduce_kernel<true, true>), rgrid, rblock, 0, st, job.part, P, job.d, nch, b2, b2m, job.y);
        else
            hipLaunchKernelGGL((ff_decode_reduce_kernel<false, true>), rgrid, rblock, 0, st, job.part, P, job.d, nch, b2, b2m, job.y);
    } else {
        if (job.bf16)
            hipLaunchKernelGGL((ff_decode_reduce_kernel<true, false>), rgrid, rblock, 0, st, job.part, P, job.d, nch, b2, b2m, job.y);
        else
            hipLaunchKernelGGL((ff_decode_reduce_kernel<false, false>), rgrid, rblock, 0, st, job.part, P, job.d, nch, b2, b2m, job.y);
    }
    rc = check_launch("ff_decode_reduce_kernel");
    if (rc == GRIFFIN_OK && ev_end && hipEventRecord(ev_end, st) != hipSuccess)
        return set_hip_error(hipGetLastError(), "hipEventRecord");
    return rc;
}

}  // namespace griffin
