// jatam_mlp.hip - the surrogate MLP: training and inference on gfx950.
//
// Not from the paper (which has no learned part): the surrogate predicts a
// genotype's class (UNBOUND / ND / DET) and log(1 + size) from its edge
// colours, so the batched path can order work and the GA can screen
// offspring; every reported class still comes from exact assembly.
//
// x = one-hot of the 12 edge colours (12 x 8; absent tiles all zero)
// h1 = relu(x W1 + b1), h2 = relu(h1 W2 + b2) (256 wide), out = h2 W3 + b3.
// Loss = mean cross-entropy of the 3 class logits + mean squared error of
// log1p(size).  Weights are kept in fp32 (with Adam moments) and used as
// bf16; h1, h2 and the hidden gradients are stored as bf16; every product
// accumulates in fp32.
//
//   layer 1      in training a gather, the sum of 4t rows of W1; in scoring a
//                product with the one-hot input like the others
//   h1 W2, dh2 W2^T, h1^T dh2, x^T dh1
//                bf16 matrix products (v_mfma_f32_16x16x32_bf16) with bias, ReLU
//                and masks applied to the results in registers
//   head, loss   per-sample dot products of length 256 and a softmax
//   Adam         elementwise over the 91,652 fp32 parameters
//
// Operand layout of the 16x16x32 MFMA (one wave): lane l holds
//   A[l % 16][8 * (l / 16) + i], i < 8      (16 x 32, M x K)
//   B[8 * (l / 16) + i][l % 16], i < 8      (32 x 16, K x N)
// and receives D[4 * (l / 16) + i][l % 16], i < 4.
#include "jatam_device.hpp"
#include "jatam_internal.hpp"

namespace jatam {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

// fp32 -> bf16, round to nearest even (NaN kept quiet).
__device__ __forceinline__ uint16_t bf16_bits(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u)
        return (uint16_t)((u >> 16) | 0x40u);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ float bf16_float(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Element (n, k) of a weight operand of K k's in the order of the matrix cores'
// loads: blocks of 16 n x 32 k (1 KB), lane n % 16 + 16 (k % 32 / 8) of a block
// with 8 k's.
__device__ __forceinline__ int weight_at(int n, int k, int K)
{
    return ((n / 16) * (K / 32) + k / 32) * 512 + (k % 32 / 8 * 16 + n % 16) * 8 + k % 8;
}

// Keeps the bf16 copies of weight i (flat index) equal to its fp32 master: W1
// as rows (w1b), W1, W2 and its transpose as operands (w1t, w2t: n the hidden
// unit, k the input; w2b the other way round), W3 as it is (w3b) and transposed
// (w3t[k][j] = W3[j][k]; rows 4..15 stay zero).
__device__ __forceinline__ void refresh_bf16(const MlpArgs& a, int i, float w)
{
    const uint16_t b = bf16_bits(w);
    if (i < kMlpOffB1) {
        a.w1b[i] = b;
        a.w1t[weight_at(i % kMlpHidden, i / kMlpHidden, kMlpIn)] = b;
    } else if (i >= kMlpOffW2 && i < kMlpOffB2) {
        const int r = i - kMlpOffW2;
        a.w2t[weight_at(r % kMlpHidden, r / kMlpHidden, kMlpHidden)] = b;
        a.w2b[weight_at(r / kMlpHidden, r % kMlpHidden, kMlpHidden)] = b;
    } else if (i >= kMlpOffW3 && i < kMlpOffB3) {
        const int r = i - kMlpOffW3;
        a.w3b[r] = b;
        a.w3t[(r % kMlpOut) * kMlpHidden + r / kMlpOut] = b;
    }
}

// Tiles the network reads of a genome of t tiles: the input has 12 edge slots
// (3 tiles), so a t outside 1..3 is read as no tiles at all (zero input).
__device__ __forceinline__ int mlp_tiles(int t) { return t >= 1 && t <= 3 ? t : 0; }

// ---------------------------------------------------------------------------
// Scoring in one pass: a wave takes 16 NB samples through the whole network by
// itself, W2 (128 KB) and the first 64 rows of W1 staged in LDS once a launch in
// the order the matrix cores take them.  The one-hot input is a matrix like any
// other, built in registers.  Every product is computed transposed, features x
// samples, so a lane's four results are consecutive features of one sample:
// bias, ReLU and rounding to bf16 by pairs, and two lane swaps make them the next
// product's B operand.  Activations stay in registers, and the loop has no
// barrier and writes no LDS.  The head's partial products, one per 32 hidden
// features, are added in their order.
//
// Bound by the matrix cores: scores of all 2^24 two-tile genotypes take 2.13 to
// 2.22 ms.  That is 1.02 to 1.06 PFLOP/s of the 135,168 flops a genome that the
// network asks for, and 1.3 of the 172,032 that are multiplied (the one-hot input's
// zeros, and a head of 16 outputs for 4); a product of two 8192 x 8192 matrices
// reaches 1.21.  Eight waves that shared a tile of 64 samples, each with 32 hidden
// columns and their weights in registers, took 6.26 ms, most of it rounding to bf16
// in integer steps, LDS writes of single values and two barriers a tile.  (Same
// rounding points and k order: the same bits.)
//
// NB: more samples a wave mean fewer LDS reads per product, and fewer waves with
// work.  Two-tile genomes, NB = 1 / 2 / 4, in the first form of this kernel: 32,768 of
// them 12.1 / 12.7 / 17.3 us, 65,536 18.5 / 16.4 / 18.0, 131,072 30.2 / 26.1 / 24.8,
// 2^24 3.09 / 2.59 / 2.41 ms; now, by the rule, 11.3, 15.7, 24.0 us and 2.2 ms.  So
// NB rises once every wave of the chip has 16 samples, and again at 32.
// ---------------------------------------------------------------------------
constexpr int kScoreWaves = 8;

__device__ __forceinline__ bf16x8 load_bf16x8(const uint16_t* p)
{
    return *reinterpret_cast<const bf16x8*>(p);
}

// One-hot A operand of k block kb for a genome: lane group q = l / 16 holds
// edge e = 4 kb + q, so its 8 values are 1.0 at that edge's colour (none if
// the edge is absent).
__device__ __forceinline__ bf16x8 onehot_operand(uint64_t g, int t, int bits, uint32_t cmask,
                                                 int e)
{
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if (e < 4 * t) {
        const uint32_t colour = (uint32_t)(g >> (bits * (4 * t - 1 - e))) & cmask;
        // colour < 8 for every c the network takes (its input has 8 slots per edge)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            w[q] = (colour == 2u * q ? 0x3F80u : 0u) | (colour == 2u * q + 1u ? 0x3F800000u : 0u);
    }
    bf16x8 v;
    __builtin_memcpy(&v, w, sizeof(v));
    return v;
}

typedef __attribute__((__vector_size__(2 * sizeof(float)))) float floatx2;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

// Two non-negative floats as bf16, rounded to nearest even.
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi)
{
    const bf16x2 v = __builtin_convertvector((floatx2{lo, hi}), bf16x2);
    uint32_t u;
    __builtin_memcpy(&u, &v, sizeof(u));
    return u;
}

// With 16 lanes a row and values a, b of four rows each: rows (a0, b0, a2, b2)
// and (a1, b1, a3, b3); rows (a0, a1, b0, b1) and (a2, a3, b2, b3).
__device__ __forceinline__ void swap_rows16(uint32_t& a, uint32_t& b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

__device__ __forceinline__ void swap_rows32(uint32_t& a, uint32_t& b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// Results of 32 features x 16 samples (two MFMA blocks: a lane of row q holds
// features 4q + i and 16 + 4q + i of its sample) plus bias, ReLU, as bf16: the B
// operand of a 32-feature k block (features 8q + i).
__device__ __forceinline__ bf16x8 relu_operand(const floatx4& z0, const floatx4& z1,
                                               const float4& b0, const float4& b1)
{
    uint32_t p0 = bf16_pair(fmaxf(z0[0] + b0.x, 0.f), fmaxf(z0[1] + b0.y, 0.f));
    uint32_t p1 = bf16_pair(fmaxf(z0[2] + b0.z, 0.f), fmaxf(z0[3] + b0.w, 0.f));
    uint32_t r0 = bf16_pair(fmaxf(z1[0] + b1.x, 0.f), fmaxf(z1[1] + b1.y, 0.f));
    uint32_t r1 = bf16_pair(fmaxf(z1[2] + b1.z, 0.f), fmaxf(z1[3] + b1.w, 0.f));
    swap_rows32(p0, r0);
    swap_rows16(p0, r0);
    swap_rows32(p1, r1);
    swap_rows16(p1, r1);
    const uint32_t w[4] = {p0, p1, r0, r1};
    bf16x8 v;
    __builtin_memcpy(&v, w, sizeof(v));
    return v;
}

__device__ __forceinline__ float score_of(float o0, float o1, float o2, float o3, int kind)
{
    const float mx = fmaxf(o0, fmaxf(o1, o2));
    const float e0 = expf(o0 - mx), e1 = expf(o1 - mx), e2 = expf(o2 - mx);
    const float inv = 1.f / (e0 + e1 + e2);
    return kind == JATAM_PREDICT_COST        ? expf(o3) - 1.f
           : kind == JATAM_PREDICT_P_UNBOUND ? e0 * inv
                                             : e2 * inv * expf(o3) - 1.f;
}

// kind: JATAM_PREDICT_SCREEN, _COST or _P_UNBOUND (what is written per genome);
// KB1: k blocks of 32 inputs that can be nonzero.
template <int KB1, int NB>
__global__ __launch_bounds__(512) void mlp_score_kernel(MlpArgs a, const uint64_t* genomes,
                                                               const uint8_t* tvec, int t_all,
                                                               uint32_t n, float* scores, int kind)
{
    constexpr int kW1 = KB1 < 2 ? KB1 : 2;   // k blocks of W1 in LDS (a third does not fit)
    constexpr int kHalf = NB < 2 ? NB : 2;   // sample blocks of a pass of layer 1
    constexpr uint32_t kRows = 16 * NB;
    // [32 features][k block][half of the features][lane]
    __shared__ bf16x8 w2s[8 * 8 * 2 * 64];
    __shared__ bf16x8 w1s[8 * kW1 * 2 * 64];
    const int tid = (int)threadIdx.x, wave = tid >> 6, l = tid & 63;
    const int r16 = l & 15, q = l >> 4;
    const uint32_t cmask = (uint32_t)a.c - 1u;
    for (int f = wave; f < 8 * 8 * 2; f += kScoreWaves)
        w2s[f * 64 + l] =
            load_bf16x8(a.w2t + ((2 * (f >> 4) + (f & 1)) * 8 + ((f >> 1) & 7)) * 512 + 8 * l);
    for (int f = wave; f < 8 * kW1 * 2; f += kScoreWaves)
        w1s[f * 64 + l] = load_bf16x8(
            a.w1t + ((2 * (f / (2 * kW1)) + (f & 1)) * 3 + (f >> 1) % kW1) * 512 + 8 * l);
    __syncthreads();
    const float b3v[4] = {a.p.b3[0], a.p.b3[1], a.p.b3[2], a.p.b3[3]};
    const uint32_t tiles = (n + kRows - 1) / kRows;
    const uint32_t stride = kScoreWaves * gridDim.x;
    uint32_t tile = (uint32_t)wave * gridDim.x + blockIdx.x;
    // the genome and tile count of sample l of a tile, loaded a tile ahead
    uint64_t next_g = 0;
    int next_t = 0;
    auto fetch = [&](uint32_t of) {
        const uint32_t sidx = of * kRows + (uint32_t)l % kRows;
        next_g = 0;
        next_t = 0;
        if (of < tiles && sidx < n) {
            next_g = genomes[sidx];
            next_t = mlp_tiles(tvec != nullptr ? tvec[sidx] : t_all);
        }
    };
    fetch(tile);
    for (; tile < tiles; tile += stride) {
        const uint64_t own_g = next_g;
        const int own_t = next_t;
        fetch(tile + stride < tile ? tiles : tile + stride);
        // -- layer 1, kHalf sample blocks at a time ---------------------------------
        bf16x8 h1[NB][8];
#pragma unroll
        for (int n0 = 0; n0 < NB; n0 += kHalf) {
            // the one-hot input, as B operands: row q holds edge 4 kb + q
            bf16x8 x[kHalf][KB1];
#pragma unroll
            for (int nb = 0; nb < kHalf; ++nb) {
                const int from = 16 * (n0 + nb) + r16;
                const uint64_t g = ((uint64_t)(uint32_t)__shfl((int)(own_g >> 32), from) << 32) |
                                   (uint32_t)__shfl((int)(uint32_t)own_g, from);
                const int t = __shfl(own_t, from);
#pragma unroll
                for (int kb = 0; kb < KB1; ++kb)
                    x[nb][kb] = onehot_operand(g, t, a.bits, cmask, 4 * kb + q);
            }
#pragma unroll
            for (int fb = 0; fb < 8; ++fb) {
                floatx4 acc[2][kHalf];
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int nb = 0; nb < kHalf; ++nb)
                        acc[m][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
                const float4 b0 = *reinterpret_cast<const float4*>(a.p.b1 + 32 * fb + 4 * q);
                const float4 b1 = *reinterpret_cast<const float4*>(a.p.b1 + 32 * fb + 16 + 4 * q);
#pragma unroll
                for (int kb = 0; kb < KB1; ++kb)
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        const bf16x8 w =
                            kb < kW1 ? w1s[((fb * kW1 + kb) * 2 + m) * 64 + l]
                                     : load_bf16x8(a.w1t + ((2 * fb + m) * 3 + kb) * 512 + 8 * l);
#pragma unroll
                        for (int nb = 0; nb < kHalf; ++nb)
                            acc[m][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                w, x[nb][kb], acc[m][nb], 0, 0, 0);
                    }
#pragma unroll
                for (int nb = 0; nb < kHalf; ++nb)
                    h1[n0 + nb][fb] = relu_operand(acc[0][nb], acc[1][nb], b0, b1);
                if (fb & 1)
                    __builtin_amdgcn_sched_barrier(0);
            }
        }
        // -- layer 2 and the head, 32 hidden features at a time ---------------------
        floatx4 out[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            out[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
        const bf16x8* w = w2s + l;
        bf16x8 w0 = w[0], w1 = w[64];
#pragma unroll 1
        for (int fb = 0; fb < 8; ++fb) {
            floatx4 acc[2][NB];
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[m][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
            const float4 b0 = *reinterpret_cast<const float4*>(a.p.b2 + 32 * fb + 4 * q);
            const float4 b1 = *reinterpret_cast<const float4*>(a.p.b2 + 32 * fb + 16 + 4 * q);
            const bf16x8 w3 = load_bf16x8(a.w3t + (size_t)r16 * kMlpHidden + 32 * fb + 8 * q);
#pragma unroll
            for (int kb = 0; kb < 8; ++kb) {
                // the next k block's operands on their way (the last one's: the next
                // features', or past the end the first ones again)
                w = kb == 7 && fb == 7 ? w2s + l : w + 128;
                const bf16x8 v0 = w[0], v1 = w[64];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[0][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, h1[nb][kb],
                                                                         acc[0][nb], 0, 0, 0);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[1][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, h1[nb][kb],
                                                                         acc[1][nb], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                w0 = v0;
                w1 = v1;
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const bf16x8 h2 = relu_operand(acc[0][nb], acc[1][nb], b0, b1);
                // a partial per 32 features, added in their order
                out[nb] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    w3, h2, floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            }
        }
        // -- the four outputs of sample r16 of block nb are row 0's: to row nb -----
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t v[4];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
                v[nb] = __float_as_uint(out[nb < NB ? nb : 0][i]);
            if constexpr (NB > 1)
                swap_rows16(v[0], v[1]);
            if constexpr (NB > 2) {
                swap_rows16(v[2], v[3]);
                swap_rows32(v[0], v[2]);
            }
            o[i] = __uint_as_float(v[0]) + b3v[i];
        }
        const uint32_t sidx = tile * kRows + (uint32_t)l;
        if (l < (int)kRows && sidx < n)
            scores[sidx] = score_of(o[0], o[1], o[2], o[3], kind);
    }
}

// ---------------------------------------------------------------------------
// Training and the plain forward pass.  A step of 4,096 samples is 2 GFLOP, a
// few microseconds of the matrix cores, so what bounds it is latency: launches,
// and the chains of loads and sums in each.  Twenty kernels, one per layer and
// gradient, took 239 us; now three, 34 us:
//   samples     forward, loss and the gradients of the activations, sixteen
//               samples a workgroup, everything between the layers in LDS (17 us)
//   gradients   the products over the batch, split across it, and the chunk
//               sums of the head and the biases, side by side (14 us)
//   update      the splits and chunks of each parameter added, Adam, and the
//               bf16 copies (4 us)
// Every sum keeps a fixed order, so a step has one result.
//
// Activations and their gradients go between the kernels in the order of the
// matrix cores' operands: [32 samples][16 features] blocks of 1 KB, in which
// lane (feature % 16) + 16 (sample % 32 / 8) holds 8 samples of one feature.
// ---------------------------------------------------------------------------
constexpr int kSampleRows = 16;
constexpr int kRowPitch = kMlpHidden + 8;   // bf16 of an LDS row: 16-lane reads conflict-free

__device__ __forceinline__ size_t operand_at(uint32_t sample, int feature, int features)
{
    return ((size_t)(sample / 32) * (features / 16) + feature / 16) * 512 +
           (sample % 32 / 8 * 16 + feature % 16) * 8 + sample % 8;
}

// Eight bf16 (16 bytes).
__device__ __forceinline__ uint4 pack8(const uint16_t* v)
{
    uint4 u;
    __builtin_memcpy(&u, v, sizeof(u));
    return u;
}

// Samples 16 blockIdx.x ..: with kTrain the loss, dout and the operands of the
// batch products, from n on as zeros (n_pad, a multiple of 32, rows are
// written); else out4.
//
// Wave w owns hidden columns 32w .. 32w + 31 of both products and loads its
// slices of W2 at the start, behind layer 1: with one tile a workgroup the
// weights (256 KB a workgroup, from L2) are most of its traffic (in rows instead
// of operand order they took 6 us more).  Layer 1 is a
// gather, the sum of 4t rows of W1, a sample and 8 columns a thread.  Sixteen
// rows, the matrix cores' least, give 4,096 samples a workgroup on each CU.
template <bool kTrain>
__global__ __launch_bounds__(512) void mlp_sample_kernel(MlpArgs a, const uint64_t* genomes,
                                                         const uint8_t* tvec, int t_all,
                                                         uint32_t n, const jatam_result_t* labels,
                                                         float* out4)
{
    __shared__ __attribute__((aligned(16))) uint16_t h1s[kSampleRows][kRowPitch];
    __shared__ __attribute__((aligned(16))) uint16_t h2s[kSampleRows][kRowPitch];   // then dh2
    __shared__ __attribute__((aligned(16))) float w3s[kMlpOut][kMlpHidden + 4];
    __shared__ __attribute__((aligned(16))) float douts[kSampleRows][kMlpOut];
    __shared__ uint64_t gs[kSampleRows];
    __shared__ int ts[kSampleRows];
    const int tid = (int)threadIdx.x, wave = tid >> 6, l = tid & 63;
    const int r16 = l & 15, q = l >> 4, col0 = 32 * wave;
    const uint32_t s0 = blockIdx.x * kSampleRows;
    // Everything the workgroup needs from memory is asked for at the start, in the
    // order of its use (waits are in that order): one round trip instead of six.
    // a thread's sample and 8 columns of layer 1
    const int row = tid >> 5, c8 = (tid & 31) * 8;
    const bool real = s0 + (uint32_t)row < n;
    const uint32_t cmask = (uint32_t)a.c - 1u;
    uint64_t genome = 0;
    int tiles = 0;
    if (real) {
        genome = genomes[s0 + row];
        tiles = mlp_tiles(tvec != nullptr ? tvec[s0 + row] : t_all);
    }
    const float4 b1a = *reinterpret_cast<const float4*>(a.p.b1 + c8);
    const float4 b1b = *reinterpret_cast<const float4*>(a.p.b1 + c8 + 4);
    uint4 w1[kMlpEdges];   // its rows of W1 (of an edge that is absent: some row)
#pragma unroll
    for (int e = 0; e < kMlpEdges; ++e) {
        const int shift = a.bits * max(4 * tiles - 1 - e, 0);
        const uint32_t colour = (uint32_t)(genome >> shift) & cmask;
        w1[e] = *reinterpret_cast<const uint4*>(a.w1b + (size_t)(e * 8 + colour) * kMlpHidden + c8);
    }
    __builtin_amdgcn_sched_barrier(0);
    const float b2v[2] = {a.p.b2[col0 + r16], a.p.b2[col0 + 16 + r16]};
    const uint64_t w3v = tid < kMlpHidden ? reinterpret_cast<const uint64_t*>(a.w3b)[tid] : 0;
    const float b3v = a.p.b3[l & 3];
    jatam_result_t label{JATAM_INVALID, 0, 0u, 0};
    if (kTrain && wave == 0 && s0 + (uint32_t)(l >> 2) < n)
        label = labels[s0 + (uint32_t)(l >> 2)];
    bf16x8 w2f[8][2], w2r[kTrain ? 8 : 1][2];
#pragma unroll
    for (int kb = 0; kb < 8; ++kb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
            w2f[kb][nb] = load_bf16x8(a.w2t + ((2 * wave + nb) * 8 + kb) * 512 + 8 * l);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kTrain)
#pragma unroll
        for (int kb = 0; kb < 8; ++kb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                w2r[kb][nb] = load_bf16x8(a.w2b + ((2 * wave + nb) * 8 + kb) * 512 + 8 * l);
    __builtin_amdgcn_sched_barrier(0);
    // -- layer 1 -------------------------------------------------------------------
    {
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < kMlpEdges; ++e) {
            const uint32_t ww[4] = {w1[e].x, w1[e].y, w1[e].z, w1[e].w};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float sum = acc[i] + bf16_float((uint16_t)(ww[i >> 1] >> (16 * (i & 1))));
                acc[i] = e < 4 * tiles ? sum : acc[i];
            }
        }
        const float b1v[8] = {b1a.x, b1a.y, b1a.z, b1a.w, b1b.x, b1b.y, b1b.z, b1b.w};
        uint16_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float z = acc[i] + b1v[i];
            v[i] = real && z > 0.f ? bf16_bits(z) : (uint16_t)0;   // +0, never -0
        }
        *reinterpret_cast<uint4*>(&h1s[row][c8]) = pack8(v);
    }
    if (kTrain && (tid & 31) == 0) {
        gs[row] = genome;
        ts[row] = tiles;   // none past the samples' end
    }
    if (tid < kMlpHidden)
#pragma unroll
        for (int k = 0; k < kMlpOut; ++k)
            w3s[k][tid] = bf16_float((uint16_t)(w3v >> (16 * k)));
    __syncthreads();
    // eight samples of one feature as the batch products take them
    const int feature = tid & 255, half = 8 * (tid >> 8);
    if constexpr (kTrain) {
        uint16_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            v[i] = h1s[half + i][feature];
        *reinterpret_cast<uint4*>(a.h1 + operand_at(s0 + half, feature, kMlpHidden)) = pack8(v);
        if (feature < kMlpIn) {
            const int e = feature >> 3;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int shift = a.bits * max(4 * ts[half + i] - 1 - e, 0);
                const uint32_t colour = (uint32_t)(gs[half + i] >> shift) & cmask;
                v[i] = e < 4 * ts[half + i] && colour == (uint32_t)(feature & 7) ? 0x3F80u : 0u;
            }
            *reinterpret_cast<uint4*>(a.x + operand_at(s0 + half, feature, kMlpIn)) = pack8(v);
        }
    }
    // -- layer 2: samples x features, a lane with samples 4q + i of feature r16 ---
    floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
        const bf16x8 af = load_bf16x8(&h1s[r16][32 * kb + 8 * q]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, w2f[kb][nb], acc[nb], 0, 0, 0);
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int col = col0 + 16 * nb + r16;
        uint16_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float z = acc[nb][i] + b2v[nb];
            v[i] = bf16_bits(z > 0.f ? z : 0.f);
            h2s[4 * q + i][col] = v[i];
        }
        if constexpr (kTrain)
            __builtin_memcpy(a.h2 + operand_at(s0 + 4 * q, col, kMlpHidden), v, sizeof(v));
    }
    __syncthreads();
    // -- head and loss: a lane per output, its sum in the order of the features ---
    if (wave == 0) {
        const int s = l >> 2, k = l & 3;
        const uint32_t b = s0 + (uint32_t)s;
        float o = b3v;
#pragma unroll 4
        for (int j = 0; j < kMlpHidden; j += 8) {
            const uint4 h = *reinterpret_cast<const uint4*>(&h2s[s][j]);
            const uint32_t hw[4] = {h.x, h.y, h.z, h.w};
            const float4 wa = *reinterpret_cast<const float4*>(&w3s[k][j]);
            const float4 wb = *reinterpret_cast<const float4*>(&w3s[k][j + 4]);
            const float w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
#pragma unroll
            for (int i = 0; i < 8; ++i)
                o = fmaf(bf16_float((uint16_t)(hw[i >> 1] >> (16 * (i & 1)))), w[i], o);
        }
        if (b < n && out4 != nullptr)
            out4[(size_t)b * kMlpOut + k] = o;
        if constexpr (kTrain) {
            const float o0 = __shfl(o, (l & ~3) + 0), o1 = __shfl(o, (l & ~3) + 1);
            const float o2 = __shfl(o, (l & ~3) + 2), o3 = __shfl(o, (l & ~3) + 3);
            float d = 0.f;
            if (b < n) {
                const int y = label.cls == JATAM_UNBOUND ? 0 : label.cls == JATAM_DET ? 2 : 1;
                const float mx = fmaxf(o0, fmaxf(o1, o2));
                const float e0 = expf(o0 - mx), e1 = expf(o1 - mx), e2 = expf(o2 - mx);
                const float sum = e0 + e1 + e2;
                const float py = (y == 0 ? e0 : y == 1 ? e1 : e2) / sum;
                const float err = o3 - log1pf((float)label.size);
                const float inv = 1.f / (float)n;
                if (k == 0)
                    a.loss[b] = -logf(py) + err * err;
                d = k == 3 ? 2.f * err * inv
                           : ((k == 0 ? e0 : k == 1 ? e1 : e2) / sum - (y == k ? 1.f : 0.f)) * inv;
                a.dout[(size_t)b * kMlpOut + k] = d;
            }
            douts[s][k] = d;
        }
    }
    if constexpr (!kTrain)
        return;
    __syncthreads();
    // -- dh2 = bf16((dout W3^T) * (h2 > 0)), over h2 in LDS ------------------------
    {
        uint16_t v[8];
        const float4 d = *reinterpret_cast<const float4*>(&douts[row][0]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float z = fmaf(d.x, w3s[0][c8 + i], 0.f);
            z = fmaf(d.y, w3s[1][c8 + i], z);
            z = fmaf(d.z, w3s[2][c8 + i], z);
            z = fmaf(d.w, w3s[3][c8 + i], z);
            v[i] = real && h2s[row][c8 + i] != 0 ? bf16_bits(z) : (uint16_t)0;
        }
        *reinterpret_cast<uint4*>(&h2s[row][c8]) = pack8(v);
    }
    __syncthreads();
    {
        uint16_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            v[i] = h2s[half + i][feature];
        *reinterpret_cast<uint4*>(a.dh2 + operand_at(s0 + half, feature, kMlpHidden)) = pack8(v);
    }
    // -- dh1 = bf16((dh2 W2^T) * (h1 > 0)) ------------------------------------------
    acc[0] = acc[1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < (kTrain ? 8 : 1); ++kb) {
        const bf16x8 af = load_bf16x8(&h2s[r16][32 * kb + 8 * q]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, w2r[kb][nb], acc[nb], 0, 0, 0);
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int col = col0 + 16 * nb + r16;
        uint16_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            v[i] = bf16_bits(h1s[4 * q + i][col] != 0 ? acc[nb][i] : 0.f);
        __builtin_memcpy(a.dh1 + operand_at(s0 + 4 * q, col, kMlpHidden), v, sizeof(v));
    }
}

// Row chunks of the head's and the biases' batch sums: partial sums per chunk,
// added in chunk order.
constexpr int kRedRows = 128;
constexpr int kGradTiles = (kMlpHidden / 32) * (kMlpHidden / 32) + (kMlpIn / 32) * (kMlpHidden / 32);

// Where the batch products' and sums' parts lie in MlpArgs::partial.
struct GradParts {
    int splits, chunks;
    float *w2, *w1, *w3, *b2, *b1, *b3, *loss;
};

constexpr int kMaxSplits = 16;

static GradParts grad_parts(float* base, uint32_t n, uint32_t n_pad)
{
    GradParts g;
    const int want = (int)(n_pad / 256);
    g.splits = want < 1 ? 1 : want > kMaxSplits ? kMaxSplits : want;
    g.chunks = (int)((n + kRedRows - 1) / kRedRows);
    g.w2 = base;
    g.w1 = g.w2 + (size_t)kMaxSplits * kMlpHidden * kMlpHidden;
    g.w3 = g.w1 + (size_t)kMaxSplits * kMlpIn * kMlpHidden;
    g.b2 = g.w3 + (size_t)g.chunks * kMlpHidden * kMlpOut;
    g.b1 = g.b2 + (size_t)g.chunks * kMlpHidden;
    g.b3 = g.b1 + (size_t)g.chunks * kMlpHidden;
    g.loss = g.b3 + (size_t)g.chunks * kMlpOut;
    return g;
}

size_t mlp_partial_floats(size_t max_batch)
{
    const size_t chunks = (max_batch + kRedRows - 1) / kRedRows;
    return (size_t)kMaxSplits * (kMlpHidden + kMlpIn) * kMlpHidden +
           chunks * (kMlpHidden * kMlpOut + 2 * kMlpHidden + kMlpOut + 1);
}

// Batch sums of feature j's values over chunk rows: f(row, value) in row order.
template <class F>
__device__ __forceinline__ void each_row(const uint16_t* src, uint32_t b0, uint32_t rows, int j, F f)
{
    // 128 rows of one feature are 16 reads of 16 bytes, all under way at once
    uint4 v[kRedRows / 8];
#pragma unroll
    for (int r = 0; r < kRedRows / 8; ++r)
        if ((uint32_t)(8 * r) < rows)
            v[r] = *reinterpret_cast<const uint4*>(src + operand_at(b0 + 8 * r, j, kMlpHidden));
#pragma unroll
    for (int r = 0; r < kRedRows / 8; ++r) {
        const uint32_t w[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if ((uint32_t)(8 * r + i) < rows)
                f(8 * r + i, bf16_float((uint16_t)(w[i >> 1] >> (16 * (i & 1)))));
    }
}

// dW2 = h1^T dh2 and dW1 = x^T dh1, a 32 x 32 tile and a split of the batch per
// wave, its operands straight from memory; from block `products` on, the chunk
// sums: dW3, db3 and the loss, then db2, then db1.
__global__ __launch_bounds__(256) void mlp_grad_kernel(MlpArgs a, GradParts g, uint32_t n,
                                                       uint32_t n_pad, uint32_t products)
{
    const int tid = (int)threadIdx.x, l = tid & 63;
    if (blockIdx.x < products) {
        const uint32_t task = blockIdx.x * 4 + (uint32_t)(tid >> 6);
        const uint32_t split = task / kGradTiles;
        int tile = (int)(task % kGradTiles);
        constexpr int kTiles2 = (kMlpHidden / 32) * (kMlpHidden / 32);
        const bool second = tile < kTiles2;
        tile -= second ? 0 : kTiles2;
        const int m = tile / (kMlpHidden / 32), c = tile % (kMlpHidden / 32);
        const uint16_t* const left = (second ? a.h1 : a.x) + (2 * m) * 512 + l * 8;
        const uint16_t* const right = (second ? a.dh2 : a.dh1) + (2 * c) * 512 + l * 8;
        const size_t lstep = (second ? kMlpHidden : kMlpIn) * 32, rstep = kMlpHidden * 32;
        const uint32_t blocks = n_pad / 32, per = (blocks + g.splits - 1) / g.splits;
        const uint32_t from = split * per, to = min(blocks, from + per);
        floatx4 acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        // eight k blocks' operands under way at once
        constexpr int kAhead = 8;
        for (uint32_t k0 = from; k0 < to; k0 += kAhead) {
            bf16x8 af[kAhead][2], bf[kAhead][2];
#pragma unroll
            for (int k = 0; k < kAhead; ++k)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const size_t kb = min(k0 + k, to - 1);
                    af[k][i] = load_bf16x8(left + kb * lstep + i * 512);
                    bf[k][i] = load_bf16x8(right + kb * rstep + i * 512);
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < kAhead; ++k)
                if (k0 + k < to)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                af[k][i], bf[k][j], acc[i][j], 0, 0, 0);
        }
        float* const out = second ? g.w2 + (size_t)split * kMlpHidden * kMlpHidden
                                  : g.w1 + (size_t)split * kMlpIn * kMlpHidden;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    out[(32 * m + 16 * i + 4 * (l >> 4) + e) * kMlpHidden + 32 * c + 16 * j +
                        (l & 15)] = acc[i][j][e];
        return;
    }
    __shared__ float4 douts[kRedRows];
    __shared__ float part[256];
    const uint32_t chunk = (blockIdx.x - products) % (uint32_t)g.chunks;
    const uint32_t what = (blockIdx.x - products) / (uint32_t)g.chunks;
    const uint32_t b0 = chunk * kRedRows;
    if (what > 0) {
        float s = 0.f;
        each_row(what == 1 ? a.dh2 : a.dh1, b0, min(n_pad - b0, (uint32_t)kRedRows), tid,
                 [&](int, float v) { s += v; });
        (what == 1 ? g.b2 : g.b1)[(size_t)chunk * kMlpHidden + tid] = s;
        return;
    }
    const uint32_t rows = min(n - b0, (uint32_t)kRedRows);
    if ((uint32_t)tid < rows)
        douts[tid] = reinterpret_cast<const float4*>(a.dout)[b0 + tid];
    part[tid] = (uint32_t)tid < rows ? a.loss[b0 + tid] : 0.f;
    __syncthreads();
    float s[kMlpOut] = {0.f, 0.f, 0.f, 0.f};
    each_row(a.h2, b0, rows, tid, [&](int r, float h) {
        const float4 d = douts[r];
        s[0] = fmaf(h, d.x, s[0]);
        s[1] = fmaf(h, d.y, s[1]);
        s[2] = fmaf(h, d.z, s[2]);
        s[3] = fmaf(h, d.w, s[3]);
    });
    reinterpret_cast<float4*>(g.w3)[(size_t)chunk * kMlpHidden + tid] =
        make_float4(s[0], s[1], s[2], s[3]);
    if (tid < kMlpOut) {
        float b = 0.f;
#pragma unroll 16
        for (uint32_t r = 0; r < rows; ++r)
            b += reinterpret_cast<const float*>(&douts[r])[tid];
        g.b3[(size_t)chunk * kMlpOut + tid] = b;
    }
    for (int off = 128; off > 0; off >>= 1) {
        if (tid < off)
            part[tid] += part[tid + off];
        __syncthreads();
    }
    if (tid == 0)
        g.loss[chunk] = part[0];
}

// Adam on a parameter; refreshes its bf16 copies.
__device__ __forceinline__ void adam_step(const MlpArgs& a, int i, float gi, float lr, float bc1,
                                          float bc2)
{
    const float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
    const float m = beta1 * a.m[i] + (1.f - beta1) * gi;
    const float v = beta2 * a.v[i] + (1.f - beta2) * gi * gi;
    a.m[i] = m;
    a.v[i] = v;
    const float w = a.p.flat[i] - lr * (m / bc1) / (sqrtf(v / bc2) + eps);
    a.p.flat[i] = w;
    refresh_bf16(a, i, w);
}

// Every parameter's gradient from its parts, in their order, and with lr > 0 an
// Adam step on it; the block past the parameters: the mean loss.
__global__ __launch_bounds__(256) void mlp_update_kernel(MlpArgs a, GradParts g, uint32_t n,
                                                         float* loss_out, float lr, float bc1,
                                                         float bc2)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x == 0 && loss_out != nullptr) {
            float s = 0.f;
#pragma unroll 16
            for (int c = 0; c < g.chunks; ++c)
                s += g.loss[c];
            loss_out[0] = s / (float)n;
        }
        return;
    }
    if (i >= kMlpParams)
        return;
    const float* part;
    int count, parts;
    if (i < kMlpOffB1) {
        part = g.w1 + i;
        count = kMlpIn * kMlpHidden;
        parts = g.splits;
    } else if (i < kMlpOffW2) {
        part = g.b1 + (i - kMlpOffB1);
        count = kMlpHidden;
        parts = g.chunks;
    } else if (i < kMlpOffB2) {
        part = g.w2 + (i - kMlpOffW2);
        count = kMlpHidden * kMlpHidden;
        parts = g.splits;
    } else if (i < kMlpOffW3) {
        part = g.b2 + (i - kMlpOffB2);
        count = kMlpHidden;
        parts = g.chunks;
    } else if (i < kMlpOffB3) {
        part = g.w3 + (i - kMlpOffW3);
        count = kMlpHidden * kMlpOut;
        parts = g.chunks;
    } else {
        part = g.b3 + (i - kMlpOffB3);
        count = kMlpOut;
        parts = g.chunks;
    }
    float s = 0.f;
#pragma unroll 16
    for (int p = 0; p < parts; ++p)
        s += part[(size_t)p * count];
    a.g.flat[i] = s;
    if (lr > 0.f)
        adam_step(a, i, s, lr, bc1, bc2);
}

// bf16 copies of all weights from the fp32 masters.
__global__ __launch_bounds__(256) void mlp_refresh_kernel(MlpArgs a)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < kMlpParams)
        refresh_bf16(a, i, a.p.flat[i]);
}

// The library's own initialisation: He-uniform weights from Philox words,
// w = (2u - 1) sqrt(6 / fan_in) with u = word / 2^32; biases zero.
__global__ __launch_bounds__(256) void mlp_init_kernel(MlpArgs a, uint32_t k0, uint32_t k1)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= kMlpParams)
        return;
    float w = 0.f;
    int fan_in = 0;
    if (i < kMlpOffB1)
        fan_in = kMlpIn;
    else if (i >= kMlpOffW2 && i < kMlpOffB2)
        fan_in = kMlpHidden;
    else if (i >= kMlpOffW3 && i < kMlpOffB3)
        fan_in = kMlpHidden;
    if (fan_in) {
        const Words4 r = philox4x32_10((uint32_t)i, 0, 0, 3u << 28, k0, k1);
        const float u = (float)(r.w[0] >> 8) * (1.f / 16777216.f);
        w = (2.f * u - 1.f) * sqrtf(6.f / (float)fan_in);
    }
    a.p.flat[i] = w;
    a.m[i] = 0.f;
    a.v[i] = 0.f;
    refresh_bf16(a, i, w);
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
int mlp_launch_init(const MlpArgs& a, uint64_t seed, hipStream_t s)
{
    hipLaunchKernelGGL(mlp_init_kernel, dim3((kMlpParams + 255) / 256), dim3(256), 0, s, a,
                       (uint32_t)seed, (uint32_t)(seed >> 32));
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

int mlp_launch_refresh(const MlpArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL(mlp_refresh_kernel, dim3((kMlpParams + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

// Outputs of n samples.
int mlp_launch_forward(const MlpArgs& a, const uint64_t* genomes, const uint8_t* tvec, int t_all,
                       uint32_t n, float* out4, hipStream_t s)
{
    hipLaunchKernelGGL(mlp_sample_kernel<false>, dim3((n + kSampleRows - 1) / kSampleRows),
                       dim3(512), 0, s, a, genomes, tvec, t_all, n,
                       (const jatam_result_t*)nullptr, out4);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

// Predictions of n samples (any n; no padding, no activations kept).
int mlp_launch_score(const MlpArgs& a, const uint64_t* genomes, const uint8_t* tvec, int t_all,
                     uint32_t n, float* scores, int kind, hipStream_t s)
{
    if (n == 0)
        return JATAM_OK;
    // k blocks of the one-hot input that can be nonzero: 4 edges per block
    const int kb1 = tvec != nullptr ? 3 : t_all;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return JATAM_E_HIP;
    // one workgroup fills a CU's LDS (NB: see the kernel)
    const uint64_t waves = (uint64_t)cus * kScoreWaves;
    const int nb = n <= 16 * waves ? 1 : n <= 32 * waves ? 2 : 4;
    const uint32_t tiles = (n + 16u * nb - 1) / (16u * nb);
    const uint32_t blocks = tiles < (uint32_t)cus ? tiles : (uint32_t)cus;
    auto launch = [&](auto one, auto two, auto four) {
        hipLaunchKernelGGL(nb == 1 ? one : nb == 2 ? two : four, dim3(blocks),
                           dim3(64 * kScoreWaves), 0, s, a, genomes, tvec, t_all, n, scores,
                           kind);
    };
    if (kb1 == 1)
        launch(mlp_score_kernel<1, 1>, mlp_score_kernel<1, 2>, mlp_score_kernel<1, 4>);
    else if (kb1 == 2)
        launch(mlp_score_kernel<2, 1>, mlp_score_kernel<2, 2>, mlp_score_kernel<2, 4>);
    else
        launch(mlp_score_kernel<3, 1>, mlp_score_kernel<3, 2>, mlp_score_kernel<3, 4>);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

// Loss and gradients of n samples, padded to n_pad (a multiple of 32) in the
// workspace; with lr > 0 Adam step number `step`.
int mlp_launch_train(const MlpArgs& a, const uint64_t* genomes, const uint8_t* tvec, int t_all,
                     const jatam_result_t* labels, uint32_t n, uint32_t n_pad, float lr, int step,
                     float* loss_out, hipStream_t s)
{
    const GradParts g = grad_parts(a.partial, n, n_pad);
    hipLaunchKernelGGL(mlp_sample_kernel<true>, dim3(n_pad / kSampleRows), dim3(512), 0, s, a,
                       genomes, tvec, t_all, n, labels, (float*)nullptr);
    const uint32_t products = (uint32_t)(kGradTiles * g.splits / 4);
    hipLaunchKernelGGL(mlp_grad_kernel, dim3(products + 3u * (uint32_t)g.chunks), dim3(256), 0, s,
                       a, g, n, n_pad, products);
    // without both of these the parameters stay as they are
    if (hipGetLastError() != hipSuccess)
        return JATAM_E_HIP;
    const float bc1 = 1.f - powf(0.9f, (float)step);
    const float bc2 = 1.f - powf(0.999f, (float)step);
    hipLaunchKernelGGL(mlp_update_kernel, dim3((kMlpParams + 255) / 256 + 1), dim3(256), 0, s, a,
                       g, n, loss_out, lr, bc1, bc2);
    return hipGetLastError() == hipSuccess ? JATAM_OK : JATAM_E_HIP;
}

}  // namespace jatam
