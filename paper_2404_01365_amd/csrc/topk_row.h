// One row's top-k by one workgroup of 1024 threads, for rows of up to TOPK_REG_KEYS scores: the body of topk_reg_kernel and of the
// kernels that carry it beside other work.
//
// One CU does all the work of a row, so what counts is the number of barriers and of latency chains between them:
//   * wave w owns a contiguous piece of the row, lane l its keys l, l + 64, ...: the loads are coalesced and go straight to registers,
//     and at the end the positions of the selected keys follow from ballots, so the indices leave in order straight from
//     the registers (a contiguous run of keys per thread sends both through LDS: 5300 + 5000 clocks for 13824 scores);
//   * the select works on rel = key - min key; the first pass counts the eleven bits below the highest set bit of
//     (max - min) in one LDS histogram of 2048 bins: the row spreads over all of them whatever exponent the scores share, the waves'
//     adds seldom meet, and the bin of the k-th largest holds a few dozen keys of an ordinary row;
//   * all places of the KPT slots are gone through without a branch per slot (with one, whose condition is uniform, 24576 scores took
//     12.9 us, not 10.2); those past the end of the row hold rel 0;
//   * a bin of at most TOPK_LIST keys is listed in LDS, and each listed key counts the keys above it (one thread a key, the
//     list read as broadcasts); a fuller bin takes another pass of eleven bits first.
// Calls back to back, us, with keys in contiguous runs per thread, sixteen histograms of 256 bins and the digits found on the list / so: 688 scores
// 6.5 / 4.1, 4096 7.6 / 4.4, 11008 10.6 / 6.4, 14336 12.4 / 7.2, 24576 18.1 / 10.3, 32768 19.5 / 12.8.  Clocks for 11008: keys and their range
// 4000, histogram 2400, its sums 1000, list 2400, ranks 1000, counts 1100, indices 2000.
#pragma once
#include "common.h"

namespace griffin {

constexpr int TOPK_THREADS = 1024, TOPK_WAVES = TOPK_THREADS / 64;
constexpr int TOPK_REG_KEYS = 32768;
constexpr int TOPK_BIN_BITS = 11, TOPK_BINS = 1 << TOPK_BIN_BITS, TOPK_LIST = 256;
static_assert(TOPK_BINS == 2 * TOPK_THREADS, "two bins a thread");

struct __attribute__((aligned(16))) TopkShared {
    uint32_t hist[TOPK_BINS];
    uint32_t list[TOPK_LIST];
    uint32_t wmin[TOPK_WAVES], wmax[TOPK_WAVES], wsum[TOPK_WAVES], wcnt[TOPK_WAVES];
    uint32_t digit, need, count, ncand, tau;
};

// unsigned order of the keys = order of the floats
__device__ __forceinline__ uint32_t order_key(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// minimum / maximum / sum over each row of 16 lanes, in every lane of the row
__device__ __forceinline__ uint32_t row16_min(uint32_t v)
{
    v = min(v, dpp_u32<0xB1>(v));
    v = min(v, dpp_u32<0x4E>(v));
    v = min(v, dpp_u32<0x141>(v));
    return min(v, dpp_u32<0x140>(v));
}
__device__ __forceinline__ uint32_t row16_max(uint32_t v)
{
    v = max(v, dpp_u32<0xB1>(v));
    v = max(v, dpp_u32<0x4E>(v));
    v = max(v, dpp_u32<0x141>(v));
    return max(v, dpp_u32<0x140>(v));
}
__device__ __forceinline__ uint32_t row16_add(uint32_t v)
{
    v += dpp_u32<0xB1>(v);
    v += dpp_u32<0x4E>(v);
    v += dpp_u32<0x141>(v);
    return v + dpp_u32<0x140>(v);
}

// inclusive prefix sum over the wavefront
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
    const int lane = threadIdx.x & 63;
    v += dpp_u32<0x111>(v);       // row_shr 1, 2, 4, 8: lanes without a source add 0
    v += dpp_u32<0x112>(v);
    v += dpp_u32<0x114>(v);
    v += dpp_u32<0x118>(v);
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 15), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 31),
                   c = (uint32_t)__builtin_amdgcn_readlane((int)v, 47);
    return v + (lane >= 16 ? a : 0u) + (lane >= 32 ? b : 0u) + (lane >= 48 ? c : 0u);
}

// `from` and the set bits of the mask below this lane
__device__ __forceinline__ uint32_t bits_below(uint64_t m, uint32_t from = 0u)
{
    return (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, from));
}

// The k largest of the row's n <= 1024 KPT scores, ties to the lower index, as ascending indices in out[0 .. k-1].
// Sixteen waves share four SIMDs, so an instruction of the loops over the keys costs sixteen clocks a slot; a branch a slot costs
// much more (231 clocks a slot for a count of four instructions), so all KPT slots are gone through, whatever n.
template <int KPT>
__device__ __forceinline__ void topk_row(TopkShared &sh, const float *row, int n, int k, int32_t *out)
{
    static_assert(KPT % 4 == 0 && KPT <= TOPK_REG_KEYS / TOPK_THREADS, "keys come in fours");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int first_key = wave * (KPT * 64);                      // of the wave
#define TOPK_IDX(j_) (first_key + (j_) * 64 + lane)               // index of this thread's key number j_
    uint32_t key[KPT];
    {
        float v[KPT];
#pragma unroll
        for (int j = 0; j < KPT; ++j)
            v[j] = row[min(TOPK_IDX(j), n - 1)];
#pragma unroll
        for (int j = 0; j < KPT; ++j)
            key[j] = order_key(v[j]);
    }
#define TOPK_SLOTS(j_) _Pragma("unroll") for (int j_ = 0; j_ < KPT; ++j_)
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;                       // (places past the end repeat keys of the row)
    TOPK_SLOTS(j) {
        kmin = min(kmin, key[j]);
        kmax = max(kmax, key[j]);
    }
    kmin = row16_min(kmin);
    kmax = row16_max(kmax);
    kmin = min(min((uint32_t)__builtin_amdgcn_readlane((int)kmin, 0), (uint32_t)__builtin_amdgcn_readlane((int)kmin, 16)),
               min((uint32_t)__builtin_amdgcn_readlane((int)kmin, 32), (uint32_t)__builtin_amdgcn_readlane((int)kmin, 48)));
    kmax = max(max((uint32_t)__builtin_amdgcn_readlane((int)kmax, 0), (uint32_t)__builtin_amdgcn_readlane((int)kmax, 16)),
               max((uint32_t)__builtin_amdgcn_readlane((int)kmax, 32), (uint32_t)__builtin_amdgcn_readlane((int)kmax, 48)));
    if (lane == 0) {
        sh.wmin[wave] = kmin;
        sh.wmax[wave] = kmax;
    }
    *(uint2 *)&sh.hist[2 * tid] = make_uint2(0u, 0u);
    if (tid < TOPK_LIST)
        sh.list[tid] = 0;
    if (tid == 0)
        sh.ncand = 0;
    __syncthreads();
    kmin = (uint32_t)__builtin_amdgcn_readfirstlane((int)row16_min(sh.wmin[lane & 15]));
    kmax = (uint32_t)__builtin_amdgcn_readfirstlane((int)row16_max(sh.wmax[lane & 15]));
    const uint32_t range = kmax - kmin;
    // rel: order and ties are those of the keys.  Places past the end get rel 0: counted along with the least keys and listed
    // with them they change no rank from above, and they come behind every key that equals them, of which there are enough.
    TOPK_SLOTS(j)
        key[j] = TOPK_IDX(j) < n ? key[j] - kmin : 0u;

    // Bits hi and up of the k-th largest rel are known: they are `pref`.  `need` of the keys that share them are still wanted;
    // `all`: and no key equal to the k-th largest is left out (not said of rel 0, which places past the end have too).
    int hi = range ? 32 - __builtin_clz(range) : 0;
    uint32_t pref = 0, need = (uint32_t)k, tau = 0;
    bool all = false;
    for (bool first = true; hi > 0; first = false) {
        const int w = min(hi, TOPK_BIN_BITS), sft = hi - w;
        // A row with many equal scores would send whole waves to one bin, one add after the other: each wave looks at its first slot once,
        // and if more than eight of its lanes share a digit there, the lanes that share the digit of a slot's first key send
        // one add with their count.  So does every wave in a pass that is not the first, where few keys take part.
        bool aggregate = !first;
        if (first) {
            const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(key[0] >> sft));
            aggregate = __builtin_popcountll(__ballot((key[0] >> sft) == d0)) > 8;
        }
        if (first_key >= n) {
            // no key of the row: neither counted nor listed
        } else if (aggregate) {
            TOPK_SLOTS(j) {
                const bool c = first || (key[j] >> (hi & 31)) == pref;
                const uint32_t digit = (key[j] >> sft) & (TOPK_BINS - 1);
                const uint64_t m = __ballot(c);
                if (m) {
                    const int leader = __builtin_ctzll(m);
                    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)digit, leader);
                    const uint64_t same = __ballot(c && digit == d0);
                    if (lane == leader)
                        atomicAdd(&sh.hist[d0], (uint32_t)__builtin_popcountll(same));
                    else if (c && digit != d0)
                        atomicAdd(&sh.hist[digit], 1u);
                }
            }
        } else if (first_key + KPT * 64 <= n) {
            TOPK_SLOTS(j)
                atomicAdd(&sh.hist[key[j] >> sft], 1u);
        } else {                               // the row ends in this wave: its places past the end in one add
            TOPK_SLOTS(j)
                if (TOPK_IDX(j) < n)
                    atomicAdd(&sh.hist[key[j] >> sft], 1u);
            if (lane == 0)
                atomicAdd(&sh.hist[0], (uint32_t)(first_key + KPT * 64 - n));
        }
        __syncthreads();
        // thread t has the bins 2047 - 2t and 2046 - 2t: `before` of the keys are in bins above them
        const uint2 h = *(const uint2 *)&sh.hist[TOPK_BINS - 2 - 2 * tid];
        const uint32_t inc = wave_scan(h.x + h.y);
        if (lane == 63)
            sh.wsum[wave] = inc;
        __syncthreads();
        const uint32_t before = row16_add((lane & 15) < wave ? sh.wsum[lane & 15] : 0u) + inc - (h.x + h.y);
        if (before < need && need <= before + h.x + h.y) {        // one thread: there are at least `need` keys
            const bool up = need <= before + h.y;
            sh.digit = (uint32_t)(TOPK_BINS - 2 - 2 * tid) + (up ? 1u : 0u);
            sh.need = need - before - (up ? 0u : h.y);
            sh.count = up ? h.y : h.x;
        }
        __syncthreads();
        pref = (pref << w) | (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.digit);
        need = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.need);
        const int count = __builtin_amdgcn_readfirstlane((int)sh.count);
        hi = sft;
        tau = pref << hi;
        if (pref > 0 && need == (uint32_t)count) {       // the whole bin: everything from its lower end on
            all = true;
            break;
        }
        if (hi > 0 && count <= TOPK_LIST) {
            const uint32_t low = (1u << hi) - 1u;
            uint32_t mine = 0;
            TOPK_SLOTS(j)
                mine += (uint32_t)__builtin_popcountll(__ballot((key[j] >> hi) == pref));
            if (mine && first_key < n) {
                uint32_t at = 0;
                if (lane == 0)
                    at = atomicAdd(&sh.ncand, mine);
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
                TOPK_SLOTS(j) {
                    const bool c = (key[j] >> hi) == pref;
                    const uint64_t m = __ballot(c);
                    if (c)
                        sh.list[at + bits_below(m)] = key[j] & low;
                    at += (uint32_t)__builtin_popcountll(m);
                }
            }
            __syncthreads();
            if (tid < count) {
                const uint32_t v = sh.list[tid];
                uint32_t above = 0, same = 0;
                for (int i = 0; i < count; i += 4) {      // entries past the end are 0: none is above, and beside v = 0, the least
                    const uint4 o = *(const uint4 *)&sh.list[i];      // there is, they only say that there are enough
                    above += (o.x > v ? 1u : 0u) + (o.y > v ? 1u : 0u) + (o.z > v ? 1u : 0u) + (o.w > v ? 1u : 0u);
                    same += (o.x == v ? 1u : 0u) + (o.y == v ? 1u : 0u) + (o.z == v ? 1u : 0u) + (o.w == v ? 1u : 0u);
                }
                if (above < need && need <= above + same) {       // all threads of that value write the same
                    sh.tau = v;
                    sh.need = need - above;
                    sh.count = same;
                }
            }
            __syncthreads();
            tau |= (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.tau);
            need = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.need);
            all = tau > 0 && need == (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.count);
            break;
        }
        if (hi > 0) {                          // another pass: the histogram was last read before the last barrier
            *(uint2 *)&sh.hist[2 * tid] = make_uint2(0u, 0u);
            __syncthreads();
        }
    }
    // tau: rel of the k-th largest score (or below it and above the next, if `all`); `need` of the keys equal to it are kept,
    // those of the lowest indices
    if (all) {
        uint32_t mine = 0;
        TOPK_SLOTS(j)
            mine += (uint32_t)__builtin_popcountll(__ballot(key[j] >= tau));
        if (lane == 0)
            sh.wcnt[wave] = mine;
        __syncthreads();
        uint32_t p = (uint32_t)__builtin_amdgcn_readfirstlane((int)row16_add((lane & 15) < wave ? sh.wcnt[lane & 15] : 0u));
        TOPK_SLOTS(j) {
            const bool c = key[j] >= tau;
            const uint64_t m = __ballot(c);
            if (c)
                out[bits_below(m, p)] = TOPK_IDX(j);
            p += (uint32_t)__builtin_popcountll(m);
        }
        return;
    }
    uint32_t c_gt = 0, c_eq = 0;
    TOPK_SLOTS(j) {
        c_gt += (uint32_t)__builtin_popcountll(__ballot(key[j] > tau));
        c_eq += (uint32_t)__builtin_popcountll(__ballot(key[j] == tau));
    }
    if (lane == 0)
        sh.wcnt[wave] = c_gt | c_eq << 16;     // each total is at most 32768
    __syncthreads();
    const uint32_t excl = (uint32_t)__builtin_amdgcn_readfirstlane((int)row16_add((lane & 15) < wave ? sh.wcnt[lane & 15] : 0u));
    uint32_t p_gt = excl & 0xFFFFu, p_eq = excl >> 16;
    TOPK_SLOTS(j) {
        const bool gt = key[j] > tau, eq = key[j] == tau;
        const uint64_t m_gt = __ballot(gt), m_eq = __ballot(eq);
        const uint32_t e = bits_below(m_eq, p_eq);
        if (gt || (eq && e < need))
            out[bits_below(m_gt, p_gt) + min(e, need)] = TOPK_IDX(j);
        p_gt += (uint32_t)__builtin_popcountll(m_gt);
        p_eq += (uint32_t)__builtin_popcountll(m_eq);
    }
#undef TOPK_SLOTS
#undef TOPK_IDX
}

// Kernels that carry the rows of a TopkJob in their first workgroups (of TOPK_THREADS threads) come in four lengths of row.
// Every workgroup of such a kernel has the registers of the longest row (128 and a spilled word for 32 scores a thread, which rows of 24576 take, too): that
// costs nothing that shows.  45 prompt phases with the top-k beside the output instead of before it, 64 to 6000 tokens and 4096 to 32768 scores, take 0.97 of the
// time (geometric mean), none more than the runs differ: 2048 tokens of 3072 x 24576 795 / 780 us, 2000 of 4096 x 32768 1325 / 1320, 64 of 512 x 24576 69 / 64.
inline bool topk_rides(const TopkJob *t) { return t && t->n <= TOPK_REG_KEYS; }
#define TOPK_RIDE(n_, GO_)                                                                            \
    {                                                                                                 \
        if ((n_) <= 4 * TOPK_THREADS) GO_(4)                                                          \
        else if ((n_) <= 8 * TOPK_THREADS) GO_(8)                                                     \
        else if ((n_) <= 16 * TOPK_THREADS) GO_(16)                                                   \
        else GO_(32)                                                                                  \
    }

}  // namespace griffin
