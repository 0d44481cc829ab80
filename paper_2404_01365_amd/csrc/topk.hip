// Expert set E (Section 4.2): indices of the k largest entries of the statistic s.
// Exact selection, ties to the lowest index, indices returned ascending.
//
// One workgroup per score row.  fp32 scores are mapped to uint32 keys whose unsigned order is
// the floats' order; a radix select over LDS histograms finds the k-th largest key tau and how
// many entries equal to tau are still needed; an ordered compaction then writes every index with
// key > tau plus the first `need` indices with key == tau, in ascending order.
// Rows of up to 32768 scores (every model shape in use) keep their keys in registers
// (topk_row.h); longer rows take four passes of eight bits with the keys in LDS (up to 36864)
// or re-read from L2 on every pass (up to 2^20), contiguous chunks of them per thread.
#include "topk_row.h"

namespace griffin {

// exclusive scan of one value per thread across the workgroup; `total` gets the sum.
// `sh` must hold TOPK_THREADS/64 + 1 entries.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *sh, uint32_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t t = __shfl_up(inc, off, 64);
        if (lane >= off)
            inc += t;
    }
    __syncthreads();            // sh may still be read from a previous call
    if (lane == 63)
        sh[wave] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int w = 0; w < TOPK_THREADS / 64; ++w) {
            uint32_t t = sh[w];
            sh[w] = run;
            run += t;
        }
        sh[TOPK_THREADS / 64] = run;
    }
    __syncthreads();
    total = sh[TOPK_THREADS / 64];
    return sh[wave] + inc - v;
}

// CACHED: the row's keys are read from global memory once (coalesced, eight loads in flight per
// thread) into LDS and every later pass works from there; without it each of the five passes
// pays the global-memory latency of its loads again, one after the other.
constexpr int TOPK_CACHE_KEYS = 36864;       // 144 KB of LDS

template <bool CACHED>
__global__ __launch_bounds__(TOPK_THREADS) void topk_select_kernel(const float *scores, int n, int k,
                                                                   int32_t *idx_out)
{
    __shared__ uint32_t keys[CACHED ? TOPK_CACHE_KEYS : 1];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t sh_digit, sh_need;
    __shared__ uint32_t sh_scan[TOPK_THREADS / 64 + 1];

    const float *row = scores + (int64_t)blockIdx.x * n;
    int32_t *out = idx_out + (int64_t)blockIdx.x * k;
    const int tid = threadIdx.x;

    if (CACHED) {
        int i = tid;
        for (; i + 7 * TOPK_THREADS < n; i += 8 * TOPK_THREADS) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = row[i + u * TOPK_THREADS];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                keys[i + u * TOPK_THREADS] = order_key(v[u]);
        }
        for (; i < n; i += TOPK_THREADS)
            keys[i] = order_key(row[i]);
        __syncthreads();
    }
#define TOPK_KEY(i_) (CACHED ? keys[i_] : order_key(row[i_]))

    uint32_t prefix = 0, mask = 0, need = (uint32_t)k;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        if (tid < 256)
            hist[tid] = 0;
        __syncthreads();
        // the statistic's values sit in a narrow range, so in the first passes most keys of a wave
        // share one digit: lanes that agree with the wave's first candidate send ONE atomic with
        // their count, the others go singly
        for (int i0 = 0; i0 < n; i0 += TOPK_THREADS) {
            const int i = i0 + tid;
            uint32_t key = 0;
            bool cand = false;
            if (i < n) {
                key = TOPK_KEY(i);
                cand = (key & mask) == prefix;
            }
            const uint32_t digit = (key >> shift) & 255u;
            const uint64_t cmask = __ballot(cand);
            if (cmask != 0) {
                const int leader = __builtin_ctzll(cmask);
                const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)digit, leader);
                const uint64_t same = __ballot(cand && digit == d0);
                if ((int)(tid & 63) == leader)
                    atomicAdd(&hist[d0], (uint32_t)__builtin_popcountll(same));
                else if (cand && digit != d0)
                    atomicAdd(&hist[digit], 1u);
            }
        }
        __syncthreads();
        // the digit of the k-th largest: the one bin b with S[b] >= need > S[b+1], S[b] = sum of the
        // bins b' >= b.  One wavefront: lane l owns bins 4l .. 4l+3, suffix sums across lanes by shuffles.
        if (tid < 64) {
            const uint32_t h0 = hist[4 * tid], h1 = hist[4 * tid + 1], h2 = hist[4 * tid + 2], h3 = hist[4 * tid + 3];
            const uint32_t loc = h0 + h1 + h2 + h3;
            uint32_t suf = loc;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t t = __shfl_down(suf, off, 64);
                if (tid + off < 64)
                    suf += t;
            }
            const uint32_t s4 = suf - loc, s3 = s4 + h3, s2 = s3 + h2, s1 = s2 + h1, s0 = s1 + h0;
            if (s0 >= need && s4 < need) {
                uint32_t dg, above;
                if (s3 >= need) { dg = 3; above = s4; }
                else if (s2 >= need) { dg = 2; above = s3; }
                else if (s1 >= need) { dg = 1; above = s2; }
                else { dg = 0; above = s1; }
                sh_digit = 4u * tid + dg;
                sh_need = need - above;
            }
        }
        __syncthreads();
        prefix |= sh_digit << shift;
        mask |= 255u << shift;
        need = sh_need;
        __syncthreads();
    }
    const uint32_t tau = prefix;   // key of the k-th largest score; `need` entries equal to it are kept

    // ordered compaction over contiguous per-thread chunks
    const int chunk = (n + TOPK_THREADS - 1) / TOPK_THREADS;
    const int lo = min(tid * chunk, n), hi = min(lo + chunk, n);
    uint32_t c_gt = 0, c_eq = 0;
    for (int i = lo; i < hi; ++i) {
        const uint32_t key = TOPK_KEY(i);
        c_gt += key > tau;
        c_eq += key == tau;
    }
    uint32_t tot_gt, tot_eq;
    uint32_t p_gt = block_exclusive_scan(c_gt, sh_scan, tot_gt);
    uint32_t p_eq = block_exclusive_scan(c_eq, sh_scan, tot_eq);
    for (int i = lo; i < hi; ++i) {
        const uint32_t key = TOPK_KEY(i);
        if (key > tau) {
            out[p_gt + min(p_eq, need)] = i;
            ++p_gt;
        } else if (key == tau) {
            if (p_eq < need)
                out[p_gt + p_eq] = i;
            ++p_eq;
        }
    }
#undef TOPK_KEY
}

// Rows of up to TOPK_REG_KEYS scores (topk_row.h)
template <int KPT>
__global__ __launch_bounds__(TOPK_THREADS) void topk_reg_kernel(const float *scores, int n, int k, int32_t *idx_out)
{
    __shared__ TopkShared sh;
    topk_row<KPT>(sh, scores + (int64_t)blockIdx.x * n, n, k, idx_out + (int64_t)blockIdx.x * k);
}

int launch_topk(const float *scores, int32_t n_rows, int32_t n, int32_t k, int32_t *idx, hipStream_t st)
{
    if (n <= TOPK_REG_KEYS) {
#define TOPK_GO(KPT_) case KPT_ / 4: hipLaunchKernelGGL(topk_reg_kernel<KPT_>, dim3(n_rows), dim3(TOPK_THREADS), 0, st, scores, n, k, idx); break;
        switch ((n + 4 * TOPK_THREADS - 1) / (4 * TOPK_THREADS)) {
            TOPK_GO(4) TOPK_GO(8) TOPK_GO(12) TOPK_GO(16) TOPK_GO(20) TOPK_GO(24) TOPK_GO(28) TOPK_GO(32)
        }
#undef TOPK_GO
        return check_launch("topk_reg_kernel");
    }
    if (n <= TOPK_CACHE_KEYS)
        hipLaunchKernelGGL(topk_select_kernel<true>, dim3(n_rows), dim3(TOPK_THREADS), 0, st, scores, n, k, idx);
    else
        hipLaunchKernelGGL(topk_select_kernel<false>, dim3(n_rows), dim3(TOPK_THREADS), 0, st, scores, n, k, idx);
    return check_launch("topk_select_kernel");
}

}  // namespace griffin
