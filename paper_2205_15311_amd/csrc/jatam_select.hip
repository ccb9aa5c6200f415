// jatam_select.hip - deterministic top-k selection on the device.
//
// Keeps the k of n candidates with the highest score, ties going to the
// lower index, and lists the kept indices in ascending order.  Scores become
// 32-bit keys whose ascending order is descending score (NaN last); a radix
// select finds the k-th key D; keys below D are kept, and of the keys equal to D
// the first (k - #below) by index.  Index order comes from prefix sums, so
// nothing depends on thread timing.  No host synchronisation: every pass reads
// the previous pass's state from device memory.
#include "jatam_internal.hpp"

namespace jatam {

// Ascending key order == descending score order; NaN sorts after everything.
__device__ __forceinline__ uint32_t score_key(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u)
        return 0xFFFFFFFFu;
    const uint32_t ascending = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ~ascending;
}

// Radix select of the k-th key, 11 + 11 + 10 bits, from the top.  A pass counts
// the keys that share the digits found so far; every block of the next pass finds
// the digit from the whole histogram by itself, so a pass is one launch.  The
// blocks add to one histogram of a few hot bins, so there are few of them (128
// until each has 8,192 scores: 1,024 took 10 us a pass for 262,144 scores, their
// atomics one after the other), and a block's items lie together, for the last two
// kernels' index order.
//
// 65,536 of 262,144 scores: 102 us in 18 launches, 34 in these six; 2^22 of 2^24:
// 524 and 199.
// First bit of pass p's digit.
__device__ __forceinline__ int select_shift(int p) { return p == 0 ? 21 : p == 1 ? 10 : 0; }

__device__ __forceinline__ uint32_t select_bits_above(int p)
{
    return p == 0 ? 0u : 0xFFFFFFFFu << select_shift(p - 1);
}

// Exclusive prefix sum of v over the block's 256 threads; *total receives the
// sum.  waves: LDS for four words.
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t* waves, uint32_t* total)
{
    uint32_t sum = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)sum, off);
        sum += (int)(threadIdx.x & 63) >= off ? up : 0u;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 63)
        waves[threadIdx.x >> 6] = sum;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        before += w < (int)(threadIdx.x >> 6) ? waves[w] : 0u;
        all += waves[w];
    }
    *total = all;
    return before + sum - v;
}

// What pass p finds from the histograms before it (all of the block, with the
// same result): the key's digits above pass p, and how many of the keys with
// these digits are still to take.
struct SelectFound {
    uint32_t prefix, need;
};

__device__ __forceinline__ SelectFound select_found(const uint32_t* state, uint32_t k, int passes,
                                                    uint32_t* waves, uint32_t* found)
{
    SelectFound f{0u, k};
    for (int p = 0; p < passes; ++p) {
        const uint32_t* const hist = state + p * kSelectBins + 8 * threadIdx.x;
        uint32_t c[8], sum = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            c[i] = hist[i];
            sum += c[i];
        }
        uint32_t total;
        uint32_t before = block_prefix(sum, waves, &total);
        // the thread whose bins hold the need-th key
        if (before < f.need && f.need <= before + sum) {
            uint32_t digit = 0, need = f.need - before;
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                const bool past = digit == (uint32_t)i && need > c[i];
                need -= past ? c[i] : 0u;
                digit += past ? 1u : 0u;
            }
            found[0] = (8 * threadIdx.x + digit) << select_shift(p);
            found[1] = need;
        }
        __syncthreads();
        f.prefix |= found[0];
        f.need = found[1];
        __syncthreads();
    }
    return f;
}

__global__ __launch_bounds__(256) void select_init_kernel(uint32_t* state)
{
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < kSelectPasses * kSelectBins;
         i += gridDim.x * 256)
        state[i] = 0;
}

__global__ __launch_bounds__(256) void select_hist_kernel(const float* __restrict__ score,
                                                          uint32_t n, uint32_t k, uint32_t* state,
                                                          int pass)
{
    __shared__ uint32_t hist[kSelectBins];
    __shared__ uint32_t waves[4], found[2];
    for (uint32_t i = threadIdx.x; i < kSelectBins; i += 256)
        hist[i] = 0;
    const SelectFound f = select_found(state, k, pass, waves, found);
    __syncthreads();
    const int shift = select_shift(pass);
    const uint32_t above = select_bits_above(pass);
    const SelectRange r = select_range(n, gridDim.x, blockIdx.x);
    for (uint32_t i = threadIdx.x; i < r.count; i += 256) {
        const uint32_t key = score_key(score[r.first + i]);
        if ((key & above) == f.prefix)
            atomicAdd(&hist[(key & ~above) >> shift], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kSelectBins; i += 256)
        if (hist[i] != 0)
            atomicAdd(&state[pass * kSelectBins + i], hist[i]);
}

// Keys below the k-th key D, and equal to it, per block.
__global__ __launch_bounds__(256) void select_count_kernel(const float* __restrict__ score,
                                                           uint32_t n, uint32_t k,
                                                           const uint32_t* state, uint32_t* counts)
{
    __shared__ uint32_t waves[4], found[2], c[2];
    if (threadIdx.x < 2)
        c[threadIdx.x] = 0;
    const SelectFound f = select_found(state, k, kSelectPasses, waves, found);
    __syncthreads();
    const SelectRange r = select_range(n, gridDim.x, blockIdx.x);
    uint32_t below = 0, equal = 0;
    for (uint32_t i = threadIdx.x; i < r.count; i += 256) {
        const uint32_t key = score_key(score[r.first + i]);
        below += key < f.prefix ? 1u : 0u;
        equal += key == f.prefix ? 1u : 0u;
    }
    atomicAdd(&c[0], below);
    atomicAdd(&c[1], equal);
    __syncthreads();
    if (threadIdx.x < 2)
        counts[2 * blockIdx.x + threadIdx.x] = c[threadIdx.x];
}

// Writes the kept indices at their ranks: of the keys equal to D the first
// `need`.
__global__ __launch_bounds__(256) void select_emit_kernel(const float* __restrict__ score,
                                                          uint32_t n, uint32_t k,
                                                          const uint32_t* state,
                                                          const uint32_t* counts,
                                                          uint32_t* out_idx)
{
    __shared__ uint32_t waves[4], found[2];
    const SelectFound f = select_found(state, k, kSelectPasses, waves, found);
    // what the blocks before this one hold
    uint32_t below = 0, equal = 0, total;
    for (uint32_t b = threadIdx.x; b < blockIdx.x; b += 256) {
        below += counts[2 * b];
        equal += counts[2 * b + 1];
    }
    block_prefix(below, waves, &total);
    below = total;
    block_prefix(equal, waves, &total);
    equal = total;
    const SelectRange r = select_range(n, gridDim.x, blockIdx.x);
    for (uint32_t at = 0; at < r.count; at += 256) {
        const bool mine = at + threadIdx.x < r.count;
        const uint32_t i = r.first + at + threadIdx.x;
        const uint32_t key = mine ? score_key(score[i]) : 0xFFFFFFFFu;
        const bool is_below = mine && key < f.prefix, is_equal = mine && key == f.prefix;
        // both counts of up to 256 in one sum
        const uint32_t sums = block_prefix((is_below ? 1u : 0u) | (is_equal ? 0x10000u : 0u), waves,
                                           &total);
        const uint32_t b = below + (sums & 0xFFFFu), e = equal + (sums >> 16);
        if (is_below || (is_equal && e < f.need))
            out_idx[b + min(e, f.need)] = i;
        below += total & 0xFFFFu;
        equal += total >> 16;
    }
}

int launch_select_top(const float* scores, uint32_t n, uint32_t k, uint32_t* out_idx,
                      uint32_t* state, hipStream_t s)
{
    if (k == 0 || n == 0)
        return JATAM_OK;
    // 1,024 items a block, more once there are 128, 8,192 once those have as many
    const uint32_t grid = min((n - 1u) / 1024u + 1u,
                              max(128u, min(n / 8192u, (uint32_t)kSelectMaxBlocks)));
    hipLaunchKernelGGL(select_init_kernel, dim3(4), dim3(256), 0, s, state);
    for (int pass = 0; pass < kSelectPasses; ++pass)
        hipLaunchKernelGGL(select_hist_kernel, dim3(grid), dim3(256), 0, s, scores, n, k, state,
                           pass);
    uint32_t* const counts = state + kSelectPasses * kSelectBins;
    hipLaunchKernelGGL(select_count_kernel, dim3(grid), dim3(256), 0, s, scores, n, k, state,
                       counts);
    hipLaunchKernelGGL(select_emit_kernel, dim3(grid), dim3(256), 0, s, scores, n, k, state,
                       counts, out_idx);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

// ---------------------------------------------------------------------------
// Queue order by predicted cost: a counting sort of n scores into 256
// buckets, highest cost first.  Blocks of kOrderBlock items histogram their
// buckets (bucket-major: entry b * nblocks + block), one exclusive scan of
// the histogram gives every (bucket, block) its first queue position, and
// each block scatters its items from there with LDS cursors.  Items of one
// bucket keep no particular order among themselves (the classification's
// records never depend on the queue order).
// ---------------------------------------------------------------------------
constexpr uint32_t kOrderBlock = 4096;

// Bucket of a score (expected DET size P(DET) e^pred - 1, at least -1):
// 16 log2(score + 2) clamped to 0..255, reversed so that high costs come
// first; NaN last.
__device__ __forceinline__ uint32_t cost_bucket(float score)
{
    if (!(score == score))
        return 255u;
    const float v = 16.f * __log2f(fmaxf(score, -1.f) + 2.f);
    const uint32_t q = v < 0.f ? 0u : v > 255.f ? 255u : (uint32_t)v;
    return 255u - q;
}

__global__ __launch_bounds__(256) void order_hist_kernel(const float* __restrict__ scores,
                                                         uint32_t n, uint32_t* hist)
{
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t lo = blockIdx.x * kOrderBlock, hi = min(n, lo + kOrderBlock);
    for (uint32_t i = lo + threadIdx.x; i < hi; i += 256)
        atomicAdd(&h[cost_bucket(scores[i])], 1u);
    __syncthreads();
    hist[threadIdx.x * gridDim.x + blockIdx.x] = h[threadIdx.x];
}

// In-place exclusive scan of m words, in three passes (per-1024 blocks,
// their totals, the block offsets added back).
__global__ __launch_bounds__(1024) void order_scan_block_kernel(uint32_t* x, uint32_t m,
                                                                uint32_t* sums)
{
    __shared__ uint32_t part[1024];
    const uint32_t i = blockIdx.x * 1024 + threadIdx.x;
    const uint32_t v = i < m ? x[i] : 0u;
    part[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint32_t add = (int)threadIdx.x >= off ? part[threadIdx.x - off] : 0u;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    if (i < m)
        x[i] = part[threadIdx.x] - v;
    if (threadIdx.x == 1023)
        sums[blockIdx.x] = part[1023];
}

// Exclusive scan of the block totals (one block, loops over them).
__global__ __launch_bounds__(1024) void order_scan_sums_kernel(uint32_t* sums, uint32_t nblocks)
{
    __shared__ uint32_t part[1024];
    const uint32_t per = (nblocks + 1023) / 1024;
    const uint32_t lo = threadIdx.x * per, hi = min(nblocks, lo + per);
    uint32_t s = 0;
    for (uint32_t b = lo; b < hi; ++b)
        s += sums[b];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint32_t add = (int)threadIdx.x >= off ? part[threadIdx.x - off] : 0u;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    uint32_t run = part[threadIdx.x] - s;
    for (uint32_t b = lo; b < hi; ++b) {
        const uint32_t v = sums[b];
        sums[b] = run;
        run += v;
    }
}

__global__ __launch_bounds__(1024) void order_scan_add_kernel(uint32_t* x, const uint32_t* sums,
                                                              uint32_t m)
{
    const uint32_t i = blockIdx.x * 1024 + threadIdx.x;
    if (i < m)
        x[i] += sums[blockIdx.x];
}

__global__ __launch_bounds__(256) void order_scatter_kernel(const float* __restrict__ scores,
                                                            uint32_t n, const uint32_t* hist,
                                                            uint32_t* order)
{
    __shared__ uint32_t cursor[256];
    cursor[threadIdx.x] = hist[threadIdx.x * gridDim.x + blockIdx.x];
    __syncthreads();
    const uint32_t lo = blockIdx.x * kOrderBlock, hi = min(n, lo + kOrderBlock);
    for (uint32_t i = lo + threadIdx.x; i < hi; i += 256)
        order[atomicAdd(&cursor[cost_bucket(scores[i])], 1u)] = i;
}

uint64_t order_work_words(uint64_t n)
{
    const uint64_t m = 256 * ((n + kOrderBlock - 1) / kOrderBlock);
    return m + (m + 1023) / 1024 + 1;
}

int launch_order_by_cost(const float* scores, uint32_t n, uint32_t* order, uint32_t* work,
                         hipStream_t s)
{
    if (n == 0)
        return JATAM_OK;
    const uint32_t nb = (n + kOrderBlock - 1) / kOrderBlock;
    const uint32_t m = 256 * nb;
    uint32_t* hist = work;
    uint32_t* sums = work + m;
    const uint32_t sb = (m + 1023) / 1024;
    hipLaunchKernelGGL(order_hist_kernel, dim3(nb), dim3(256), 0, s, scores, n, hist);
    hipLaunchKernelGGL(order_scan_block_kernel, dim3(sb), dim3(1024), 0, s, hist, m, sums);
    // the block totals: at most 1024 of them for n up to 2^24 items, more in
    // a second level
    if (sb > 1) {
        hipLaunchKernelGGL(order_scan_sums_kernel, dim3(1), dim3(1024), 0, s, sums, sb);
        hipLaunchKernelGGL(order_scan_add_kernel, dim3(sb), dim3(1024), 0, s, hist, sums, m);
    }
    hipLaunchKernelGGL(order_scatter_kernel, dim3(nb), dim3(256), 0, s, scores, n, hist, order);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

}  // namespace jatam
