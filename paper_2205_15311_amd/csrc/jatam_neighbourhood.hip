// jatam_neighbourhood.hip - robustness and evolvability of genotypes (§1.1).
//
// Robustness is the share of a genotype's single mutations that keep its
// phenotype, evolvability the number of different phenotypes its single
// mutations reach.  A single mutation flips one bit of the genome (the
// mutation operator flips bits, App. B.3), so a t-tile genotype has
// 4 t log2(c) single mutants.  A phenotype is UNBOUND, non-deterministic
// (either ND class) or a deterministic shape (size and D4 hash).
//
// The single mutants of a list or range of genotypes (for classification by
// any classify call); the counts from the genotypes' and their mutants'
// records; and the counts from the records of a whole space (S_{1,8},
// S_{2,8}: every mutant is a member, so its record is read at genome ^
// (1 << k), nothing is classified twice).  All integer work.
#include "jatam_internal.hpp"

namespace jatam {

// 1: UNBOUND, 2: non-deterministic, else 4 + size * 2^32 + hash (DET).
__device__ __forceinline__ uint64_t phenotype_key(const jatam_result_t& r)
{
    if (r.cls == JATAM_DET)
        return 4ull + ((uint64_t)(uint32_t)r.size << 32) + (uint64_t)r.hash;
    return r.cls == JATAM_UNBOUND ? 1ull : 2ull;
}

__global__ __launch_bounds__(256) void mutants_kernel(const uint64_t* __restrict__ genomes,
                                                      uint64_t first, uint64_t n, int nbits,
                                                      uint64_t* __restrict__ out)
{
    const uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n * (uint64_t)nbits)
        return;
    const uint64_t i = e / (uint64_t)nbits;
    const int k = (int)(e - i * (uint64_t)nbits);
    const uint64_t g = genomes != nullptr ? genomes[i] : first + i;
    out[e] = g ^ (1ull << k);
}

constexpr int kNbLanes = 64;   // one-wave blocks: 64 lanes x up to 64 keys in LDS

// Counts for a genotype, its mutants' keys already in keys[k * lanes].
__device__ __forceinline__ jatam_neighbourhood_t count_neighbourhood(const uint64_t* keys,
                                                                     uint64_t own, int nbits,
                                                                     uint32_t lanes = kNbLanes)
{
    int robust = 0, evolv = 0;
    for (int k = 0; k < nbits; ++k) {
        const uint64_t kk = keys[(uint32_t)k * lanes];
        robust += kk == own;
        bool fresh = kk != own;
        for (int j = 0; j < k && fresh; ++j)
            fresh = keys[(uint32_t)j * lanes] != kk;
        evolv += fresh;
    }
    return jatam_neighbourhood_t{robust, evolv};
}

__global__ __launch_bounds__(kNbLanes) void neighbourhood_kernel(
    const jatam_result_t* __restrict__ own, const jatam_result_t* __restrict__ mut, uint64_t n,
    int nbits, jatam_neighbourhood_t* __restrict__ out)
{
    __shared__ uint64_t keys[64 * kNbLanes];
    const uint64_t i = (uint64_t)blockIdx.x * kNbLanes + threadIdx.x;
    if (i >= n)
        return;
    uint64_t* lk = keys + threadIdx.x;
    for (int k = 0; k < nbits; ++k)
        lk[k * kNbLanes] = phenotype_key(mut[i * (uint64_t)nbits + k]);
    out[i] = count_neighbourhood(lk, phenotype_key(own[i]), nbits);
}

// ---------------------------------------------------------------------------
// A whole space's counts.
//
// A workgroup takes a window of 2^b genotypes (genome bits 0 .. b-1) and gives
// every phenotype it meets a number below 64 (a table of exact 64-bit keys in
// LDS), so a genotype's mutants are a 64-bit set: the distinct count is its
// population count.  The window's own numbers lie in LDS, one byte each: the
// mutants of bits below b are found there, four genotypes to a word, and only
// those of the other bits are read from the records, each as a stretch in the
// order of the window's own genotypes, which coalesces.
//
// Bound by those reads, (1 + bits - b) x 16 bytes a genotype through the
// caches, so b is as large as leaves a window for every compute unit (2^24
// genotypes: b = 16, 64 KB of LDS).  The windows of one XCD are neighbours and
// advance together, so of the bits above b the lowest five meet in its L2.
// One lane per genotype that gathered all of its mutants' records and
// compared their keys in pairs took 5.86 ms over S_{2,8}; this takes 0.32 ms.
// ---------------------------------------------------------------------------
constexpr int kNbSlots = 64;
constexpr uint32_t kNbLds = 1u << 16;    // bytes of LDS, a window's numbers or a recount's keys

// The number of phenotype `key` in the window's table, entered if new; `full` is
// set (and any number returned) if it has no room left.
__device__ __forceinline__ uint32_t phenotype_number(unsigned long long* table, uint64_t key,
                                                     uint32_t& full)
{
    if (key <= 2ull)
        return (uint32_t)key - 1u;   // UNBOUND, non-deterministic: entries 0 and 1
    uint32_t s = ((uint32_t)key * 0x9E3779B1u ^ (uint32_t)(key >> 32) * 0x85EBCA77u) >> 26;
    for (int probe = 0; probe < kNbSlots; ++probe, s = (s + 1) & (kNbSlots - 1)) {
        unsigned long long seen =
            __hip_atomic_load(&table[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (seen == 0ull)
            seen = atomicCAS(&table[s], 0ull, (unsigned long long)key);
        if (seen == 0ull || seen == key)
            return s;
    }
    full = 1u;
    return 0u;
}

// Four neighbouring genotypes' records.
struct Quad {
    jatam_result_t r[4];

    __device__ __forceinline__ void load(const jatam_result_t* __restrict__ p)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            r[q] = p[q];
    }
    // their phenotypes' numbers, one byte each
    __device__ __forceinline__ uint32_t numbers(unsigned long long* table, uint32_t& full) const
    {
        uint32_t v = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v |= phenotype_number(table, phenotype_key(r[q]), full) << (8 * q);
        return v;
    }
};

// Four genotypes' mutants as sets of phenotype numbers.
struct MutantSets {
    uint64_t set[4];
    uint32_t other;     // byte q: mutants with another phenotype than genotype q
    uint32_t own;       // byte q: genotype q's number

    // one mutant of each genotype, byte q the number of genotype q's
    __device__ __forceinline__ void add(uint32_t ids)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            set[q] |= 1ull << ((ids >> (8 * q)) & 63u);
        // numbers are below 64, so their XOR plus 0x7F has bit 7 iff they differ
        other += (((ids ^ own) + 0x7F7F7F7Fu) >> 7) & 0x01010101u;
    }
};

__global__ __launch_bounds__(1024) void neighbourhood_space_kernel(
    const jatam_result_t* __restrict__ space, uint64_t first, uint64_t n, int nbits, int b,
    uint64_t window0, uint32_t windows, jatam_neighbourhood_t* __restrict__ out)
{
    // 2^b numbers, four to a word (kNbLds bytes)
    extern __shared__ __attribute__((aligned(16))) uint32_t ids[];
    __shared__ unsigned long long table[kNbSlots];
    __shared__ uint32_t crowded;   // a phenotype found no room in the table
    const uint32_t tid = threadIdx.x, threads = blockDim.x;
    // workgroups go to the XCDs in turn: each XCD takes neighbouring windows
    const uint32_t per_xcd = (windows + 7u) / 8u;
    const uint32_t wi = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per_xcd || wi >= windows)
        return;   // the whole workgroup
    const uint64_t base = (window0 + wi) << b;
    for (uint32_t s = tid; s < (uint32_t)kNbSlots; s += threads)
        table[s] = s < 2u ? s + 1ull : 0ull;
    if (tid == 0)
        crowded = 0u;
    __syncthreads();
    uint32_t full = 0;
    const uint32_t words = (1u << b) / 4u;
    // records are loaded a round ahead of their lookups: the loads of one
    // round, four a lane, are what hides their own latency
    Quad next;
    next.load(space + base + 4u * (tid < words ? tid : 0u));
    for (uint32_t i = tid; i < words; i += threads) {
        const Quad cur = next;
        next.load(space + base + 4u * (i + threads < words ? i + threads : i));
        ids[i] = cur.numbers(table, full);
    }
    if (full != 0)
        crowded = 1u;
    __syncthreads();
    const uint32_t sets = crowded == 0u ? words : 0u;
    for (uint32_t i = tid; i < sets; i += threads) {
        const uint64_t g0 = base + 4u * i;
        if (g0 + 3u < first || g0 >= first + n)
            continue;
        if (b < nbits)
            next.load(space + (g0 ^ (1ull << b)));
        const uint32_t own = ids[i];
        MutantSets m{{0ull, 0ull, 0ull, 0ull}, 0u, own};
        // bits 0 and 1: the other genotypes of the word
        m.add(((own >> 8) & 0x00FF00FFu) | ((own << 8) & 0xFF00FF00u));
        m.add((own >> 16) | (own << 16));
        for (int k = 2; k < b; ++k)
            m.add(ids[i ^ (1u << (k - 2))]);
        for (int k = b; k < nbits; ++k) {
            const Quad cur = next;
            next.load(space + (g0 ^ (1ull << (k + 1 < nbits ? k + 1 : k))));
            m.add(cur.numbers(table, full));
        }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint64_t g = g0 + q;
            if (g < first || g >= first + n)
                continue;
            jatam_neighbourhood_t c;
            c.robust = nbits - (int)((m.other >> (8 * q)) & 0xFFu);
            c.evolv = __popcll(m.set[q] & ~(1ull << ((own >> (8 * q)) & 63u)));
            out[g - first] = c;
        }
    }
    if (full != 0)
        crowded = 1u;
    __syncthreads();
    if (crowded == 0u)
        return;
    // More phenotypes than the table holds: the window's counts once more, a
    // genotype a lane, its mutants' keys in LDS in place of the numbers and
    // compared in pairs.  2^24 genotypes of 200 phenotypes 6.3 ms (13 of them, which
    // the table holds, 0.28); with the pairs' records read from memory 20.3.
    uint64_t* const keys = reinterpret_cast<uint64_t*>(ids);
    const uint32_t lanes = min(threads, kNbLds / 8u / (uint32_t)nbits / 64u * 64u);
    const uint64_t last = min(first + n, base + (1ull << b));
    for (uint64_t g = max(first, base) + tid; tid < lanes && g < last; g += lanes) {
        for (int k = 0; k < nbits; ++k)
            keys[(uint32_t)k * lanes + tid] = phenotype_key(space[g ^ (1ull << k)]);
        out[g - first] = count_neighbourhood(keys + tid, phenotype_key(space[g]), nbits, lanes);
    }
}

int launch_mutants(const uint64_t* genomes, uint64_t first, int64_t n, int nbits, uint64_t* out,
                   hipStream_t s)
{
    const uint64_t total = (uint64_t)n * (uint64_t)nbits;
    for (uint64_t at = 0; at < total;) {
        // whole genotypes per launch, at most 2^31 elements
        const uint64_t per = ((1ull << 31) / (uint64_t)nbits) * (uint64_t)nbits;
        const uint64_t e = total - at < per ? total - at : per;
        const uint64_t gi = at / (uint64_t)nbits;
        hipLaunchKernelGGL(mutants_kernel, dim3((unsigned)((e + 255) / 256)), dim3(256), 0, s,
                           genomes != nullptr ? genomes + gi : nullptr, first + gi,
                           e / (uint64_t)nbits, nbits, out + at);
        at += e;
    }
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

int launch_neighbourhood(const jatam_result_t* own, const jatam_result_t* mut, int64_t n,
                         int nbits, jatam_neighbourhood_t* out, hipStream_t s)
{
    for (int64_t at = 0; at < n; at += (int64_t)1 << 30) {
        const int64_t k = n - at < ((int64_t)1 << 30) ? n - at : ((int64_t)1 << 30);
        hipLaunchKernelGGL(neighbourhood_kernel, dim3((unsigned)((k + kNbLanes - 1) / kNbLanes)),
                           dim3(kNbLanes), 0, s, own + at, mut + at * nbits, (uint64_t)k, nbits,
                           out + at);
    }
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

int launch_neighbourhood_space(const jatam_result_t* space, uint64_t first, int64_t n, int nbits,
                               jatam_neighbourhood_t* out, hipStream_t s)
{
    // windows of 2^16 genotypes (a byte each in LDS), smaller ones while they
    // would leave compute units idle; at least one thread's four genotypes.  All
    // with the LDS of the largest: of the smaller ones there are at most two a
    // compute unit, and a crowded window needs it for its keys.
    int b = nbits < 16 ? nbits : 16;
    while (b > 10 && (n >> b) < 256)
        --b;
    const uint32_t words = (1u << b) / 4u;
    const uint32_t threads = words < 64u ? 64u : words > 1024u ? 1024u : words;
    const uint64_t w0 = first >> b, w1 = (first + (uint64_t)n - 1u) >> b;
    const uint64_t per_launch = 1ull << 20;
    for (uint64_t w = w0; w <= w1; w += per_launch) {
        const uint32_t windows = (uint32_t)(w1 - w + 1u < per_launch ? w1 - w + 1u : per_launch);
        hipLaunchKernelGGL(neighbourhood_space_kernel, dim3((windows + 7u) / 8u * 8u),
                           dim3(threads), (size_t)kNbLds, s, space, first, (uint64_t)n, nbits, b,
                           w, windows, out);
    }
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

}  // namespace jatam

extern "C" {

// Bits of a genome of t tiles over c colours, or -1 if (t, c) is invalid.
static int genome_bits(int t, int c)
{
    jatam::Params p;
    return jatam::make_params(t, c, 16, 1, 1, &p) == JATAM_OK ? p.genome_bits : -1;
}

int jatam_single_mutants(const uint64_t* genotypes, uint64_t first, int64_t n, int t, int c,
                         uint64_t* mutants, void* stream)
{
    const int nbits = genome_bits(t, c);
    if (nbits < 0 || n < 0 || (n > 0 && mutants == nullptr))
        return JATAM_E_INVALID_ARG;
    if (n == 0)
        return JATAM_OK;
    if (genotypes == nullptr) {
        const uint64_t last = first + (uint64_t)(n - 1);
        if (last < first || (nbits < 64 && (last >> nbits) != 0))
            return JATAM_E_INVALID_ARG;
    }
    return jatam::launch_mutants(genotypes, first, n, nbits, mutants, (hipStream_t)stream);
}

int jatam_neighbourhood(const jatam_result_t* own, const jatam_result_t* mutant_records,
                        int64_t n, int t, int c, jatam_neighbourhood_t* out, void* stream)
{
    const int nbits = genome_bits(t, c);
    if (nbits < 0 || n < 0 ||
        (n > 0 && (own == nullptr || mutant_records == nullptr || out == nullptr)))
        return JATAM_E_INVALID_ARG;
    if (n == 0)
        return JATAM_OK;
    return jatam::launch_neighbourhood(own, mutant_records, n, nbits, out, (hipStream_t)stream);
}

int jatam_neighbourhood_space(const jatam_result_t* space, uint64_t first, int64_t n, int t,
                              int c, jatam_neighbourhood_t* out, void* stream)
{
    const int nbits = genome_bits(t, c);
    if (nbits < 0 || nbits > 32 || n < 0 || (n > 0 && (space == nullptr || out == nullptr)))
        return JATAM_E_INVALID_ARG;
    if (n == 0)
        return JATAM_OK;
    const uint64_t last = first + (uint64_t)(n - 1);
    if (last < first || (last >> nbits) != 0)
        return JATAM_E_INVALID_ARG;
    return jatam::launch_neighbourhood_space(space, first, n, nbits, out, (hipStream_t)stream);
}

}  // extern "C"
