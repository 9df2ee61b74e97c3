// Bulk hashing, first pass: most keys are settled by bfloat16 matrix instructions alone.
//
// Bulk hashing with the defined binary32 chain in layer 1 (hash_bulk.h) is bound by the binary32 matrix
// instruction (153 TFLOP/s) plus the vector instructions beside it.  A code only holds SIGNS, so this pass
// evaluates the whole network on v_mfma_f32_32x32x16_bf16 (products of bfloat16 vectors and weights are exact
// there, only the sums round differently) with the hardware's exponential, and keeps a bound on the distance of
// every output from the defined chain's.  A key all of whose outputs are further from zero than that bound has
// its code; the others (9 % of random keys at 128 -> 256 -> 128) are marked in a bitmap, and the kernels of
// hash_bulk.h hash those alone afterwards, with the chain.  The codes are the same bit for bit.
//
// The bound, in units of u = 2^-24.  One instruction adds its 16 products to c as two groups of eight,
// consecutive in k; a group's result r is within u (10 max|p| + 2 |c| + |r|) of the exact sum: nine terms and the sum of the
// products are cut at 2^-24 of the largest, then r is rounded (tests/test_gpu_hash_screen.py holds the
// instruction to it: 0.38 of that at most for one group over wide exponents, cancellation and ties, 0.49 of the sum of both for two).
//   layer 1: chain and matrix core round partial sums S_k of the same products.  With S known at k = 0 (b1), 32,
//     64, 96 and 128, |S_k| is at most the nearest of them plus the products between, so that
//       |a - a'| <= u (24 |b1| + 44 (|S_32| + |S_64| + |S_96|) + 20 |a'| + sum_j t_j |w_j x_j|),
//     t_j <= 32 (first_layer_charge).  sum_j t_j |w_j x_j| <= ||t w_i|| ||x||.
//   SiLU: |silu'(a)| <= min(1.1, 0.5 + 0.5 |a|); its two evaluations (the fixed routine, and a * rcp(1 + exp2))
//     are within 12 u |h| + 2 u |a| of each other for equal a.
//   Over all hidden units of a key that is, as norms, ||h - h'|| <= dh (see below).
//   layer 2: h' enters as hi + lo (128 u |h'|); chain and matrix core round partial sums again, charged to the nearer
//     end: |y - y'| <= u ||s w_j|| (||h'|| + dh) + ||w_j|| dh + (hidden + 16) u |y'|, s_i = second_layer_charge.
// Norms carry an absolute 1e-12, far more than any conversion or flushed term; a bound that is not a number or
// not small against the range of binary32 settles nothing.  Distances from the chain are 0.14 of their bounds at most, 0.06 but for
// wide exponents (tests/test_gpu_hash_bounds.py).
#pragma once
#include "hash_bulk.h"

namespace spotlight {
namespace screen {
using namespace hashdev;
using bulk::add_halves;
using bulk::bf16x8_t;
using bulk::f32x16_t;
using bulk::other_half;

constexpr int kWaves = 8;             // wavefronts of a workgroup
constexpr int kWords = 8;             // code words at most
constexpr int kNear = 2;              // segments of open rows that a workgroup counts in LDS
constexpr double kU = 0x1p-24;

// How often the product of index j (0 ..) of a row's `n` counts in the bounds above.
__host__ __device__ inline float first_layer_charge(int j)
{
    const int k = j % 32;   // between two known sums: the chain rounds up to 16 sums with it, the matrix core up to 2
    const int chain = k < 16 ? 16 - k : k - 16, groups = k < 8 ? 6 : k < 16 ? 3 : k < 24 ? 0 : 3;
    return static_cast<float>(chain + groups + 10);
}
__host__ __device__ inline float second_layer_charge(int i, int n)
{
    const int chain = i < n / 2 ? n / 2 - i : i - n / 2 + 1;
    return 1.75f * chain + 12.0f + 11.0f + 128.0f;  // 12 per 16 units from the groups' sums; the cut products; the split
}

// What the bound needs to know of a weight head, in front of its n_words word records.
struct LayerScale {
    float t1;         // sqrt(sum_i ||t W1_i||^2)
    float t1_max;     // max_i ||t W1_i||
    float b1;         // ||b1||
    uint32_t no_bias; // b1 is all zeros
};
struct WordScale {
    float s2;         // max_j u ||s W2_j|| over the outputs of the word
    float w2;         // max_j ||W2_j||
    uint32_t zeros;   // bit c: output c * W + word has a row of zeros (y = 0, bit 0)
    uint32_t uneven;  // its rows' bounds differ: kUneven
};
struct RowScale {     // the same of each output, in the order of the word's bits
    float s2, w2;
};
static_assert(sizeof(LayerScale) == 16 && sizeof(WordScale) == 16, "one record is 16 bytes");

constexpr float kSlack = 1e-12f;
// Rows of a word are uneven where its largest bound is in the mean more than this many times a row's own.  Equal rows stay with one
// comparison (a threshold for every output: 64 more vector instructions a tile, 9.4 -> 8.7 % open, no gain).  One row of 32 three and ten times the others, 8 heads x
// 65536, 128 -> 256 -> 128: 284 and 463 us with one bound, 238 with one for each.
constexpr float kUneven = 1.5f;

// Scales of all weight heads: [heads][1 + W] records, [heads][W][32] RowScale.
__host__ __device__ inline size_t scale_bytes(int heads, int W) { return static_cast<size_t>(heads) * ((1 + W) * 16 + W * 32 * sizeof(RowScale)); }
__device__ __forceinline__ const RowScale* row_scales(const char* scales, int heads, int whead, int W)
{
    return reinterpret_cast<const RowScale*>(scales + static_cast<int64_t>(heads) * (1 + W) * 16) + static_cast<int64_t>(whead) * W * 32;
}

// Blocks of 32 hidden units; at least two, so that the kernel below always has a next one.
__host__ __device__ inline int blocks_of(int hidden) { return hidden > 32 ? (hidden + 31) / 32 : 2; }
// Operands of a block, 64 x 16 bytes each: 8 steps of 16 k of layer 1, then [half of the block][code word] of layer 2.
__host__ __device__ constexpr int operands_of(int words) { return 8 + 2 * words; }
// Code words the kernel below is compiled for.
__host__ __device__ inline int words_for(int W) { return W <= 2 ? 2 : W <= 4 ? 4 : 8; }
constexpr int kPerBlock = 32;         // operands a workgroup of the next kernel lays out

// Lane l's part of operand f of block ub: eight weights of one row, zeros past the end.  Rows of layer 1 are
// in the order that leaves a lane of the result eight consecutive units; of layer 2, in the order of a word's bits.
__device__ __forceinline__ uint4 operand(const bf16_raw* w1, const bf16_raw* w2, int hidden, int W, int words, int ub, int f, int l)
{
    const int c = l & 31, half = l >> 5;
    if (f < 8) {
        const int unit = ub * 32 + bulk::unit_of_row(c);
        if (unit < hidden) return *reinterpret_cast<const uint4*>(w1 + static_cast<int64_t>(unit) * kHeadDim + (2 * f + half) * 8);
    } else {
        const int ks = (f - 8) / words, word = (f - 8) % words, unit = ub * 32 + ks * 16 + half * 8;
        const int j = ((c >> 3) * 4 + (c & 3) + 16 * ((c >> 2) & 1)) * W + word;
        if (unit < hidden && word < W) return *reinterpret_cast<const uint4*>(w2 + static_cast<int64_t>(j) * hidden + unit);
    }
    return make_uint4(0u, 0u, 0u, 0u);
}

// What the first pass needs of the weights.  grid (weight heads, 1 + words + ...): block 0 the norms of the first layer, block
// 1 + w those of code word w (all clear the counts of open rows); the others lay out the operands for kernels that read them again for every eight tiles (from
// the arrays as stored, a row per lane, each 16-byte load touches 64 cache lines).
// AHEAD: rows of the first layer on their way (256 hidden units: 9.2 us one at a time, 5.4 us eight).
template <int AHEAD>
__global__ __launch_bounds__(kThreads) void scales_kernel(const bf16_raw* __restrict__ w1, const bf16_raw* __restrict__ b1,
                                                          const bf16_raw* __restrict__ w2, char* __restrict__ out,
                                                          uint4* __restrict__ operands, uint32_t* __restrict__ counts, int n_counts, int hidden, int L)
{
    __shared__ float sums[kThreads / 64][3];
    __shared__ uint32_t bits[kThreads / 64];
    const int W = L / 32, whead = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = (blockIdx.y * gridDim.x + blockIdx.x) * kThreads + tid; i < n_counts; i += gridDim.x * gridDim.y * kThreads) counts[i * bulk::kCountStride] = 0;
    if (static_cast<int>(blockIdx.y) > W) {
        const int words = words_for(W), per = operands_of(words), n = blocks_of(hidden) * per;
        w1 += static_cast<int64_t>(whead) * hidden * kHeadDim;
        w2 += static_cast<int64_t>(whead) * L * hidden;
        for (int e = wave; e < kPerBlock; e += kThreads / 64) {
            const int at = (static_cast<int>(blockIdx.y) - 1 - W) * kPerBlock + e;
            if (at < n) operands[(static_cast<int64_t>(whead) * n + at) * 64 + lane] = operand(w1, w2, hidden, W, words, at / per, at % per, lane);
        }
        return;
    }
    char* rec = out + static_cast<int64_t>(whead) * (1 + W) * 16;
    float a = 0.0f, b = 0.0f, c = 0.0f;
    uint32_t any = 0;
    if (blockIdx.y == 0) {   // 16 lanes a row
        const bf16_raw* base = w1 + static_cast<int64_t>(whead) * hidden * kHeadDim;
        float charge[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) charge[e] = first_layer_charge(tid % 16 * 8 + e);
        for (int i0 = tid / 16; i0 < hidden; i0 += AHEAD * (kThreads / 16)) {
            Raw8<bf16_raw> raw[AHEAD];
#pragma unroll
            for (int p = 0; p < AHEAD; ++p) load_raw(base + static_cast<int64_t>(min(i0 + p * (kThreads / 16), hidden - 1)) * kHeadDim + tid % 16 * 8, raw[p]);
#pragma unroll
            for (int p = 0; p < AHEAD; ++p) {
                float v[8], s = 0.0f;
                expand(raw[p], v);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float t = charge[e] * v[e];
                    s = __builtin_fmaf(t, t, s);
                }
                s = bulk::add_across_16(s);             // (the lanes of a row agree on what follows)
                if (i0 + p * (kThreads / 16) < hidden) {
                    a += s;                             // 16 times, once in each lane of the row
                    b = s > b || s != s ? s : b;
                }
            }
        }
        a *= 1.0f / 16.0f;
        for (int i = tid; i < hidden; i += kThreads) {
            const float v = load1(b1 + static_cast<int64_t>(whead) * hidden + i);
            c = __builtin_fmaf(v, v, c);
            any |= __float_as_uint(v) << 1;
        }
    } else {                 // 8 lanes a row
        const int word = blockIdx.y - 1, r = tid / 8;
        const bf16_raw* row = w2 + (static_cast<int64_t>(whead) * L + r * W + word) * hidden;
#pragma unroll 4
        for (int g = tid % 8; g < hidden / 8; g += 8) {
            float v[8];
            load8(row + g * 8, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float s = second_layer_charge(g * 8 + e, hidden) * v[e];
                a = __builtin_fmaf(s, s, a);
                b = __builtin_fmaf(v[e], v[e], b);
                any |= __float_as_uint(v[e]) << 1;
            }
        }
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) {
            a += __shfl_xor(a, off);
            b += __shfl_xor(b, off);
            any |= __shfl_xor(any, off);
        }
        const float own = 1.001f * __builtin_sqrtf(b) + kSlack;
        if (tid % 8 == 0)
            const_cast<RowScale*>(row_scales(out, gridDim.x, whead, W))[word * 32 + r] = {static_cast<float>(1.001 * kU) * (__builtin_sqrtf(a) + static_cast<float>(hidden) * kSlack), own};
        c = any ? 1.0f / own : 0.0f;
#pragma unroll
        for (int off = 8; off < 64; off <<= 1) c += __shfl_xor(c, off);
    }
    // over the workgroup: sums of a and c and the largest b (layer 1), the largest a and b and the sum of c (a word); a NaN stays
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) {
        const float a2 = __shfl_xor(a, off), b2 = __shfl_xor(b, off);
        b = b2 > b || b2 != b2 ? b2 : b;
        a = blockIdx.y == 0 ? a + a2 : a2 > a || a2 != a2 ? a2 : a;
    }
    if (blockIdx.y == 0) {
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) a += __shfl_xor(a, off);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) { c += __shfl_xor(c, off); any |= __shfl_xor(any, off); }
    } else {
        // lane 8 r of a wavefront has row 8 wave + r of the word
        const unsigned long long z = __ballot(any == 0);
        any = 0;
#pragma unroll
        for (int r = 0; r < 8; ++r) any |= static_cast<uint32_t>((z >> (8 * r)) & 1) << (8 * wave + r);
    }
    if (lane == 0) { sums[wave][0] = a; sums[wave][1] = b; sums[wave][2] = c; bits[wave] = any; }
    __syncthreads();
    if (tid != 0) return;
    for (int w = 1; w < kThreads / 64; ++w) {
        const float a2 = sums[w][0], b2 = sums[w][1];
        b = b2 > b || b2 != b2 ? b2 : b;
        a = blockIdx.y == 0 ? a + a2 : a2 > a || a2 != a2 ? a2 : a;
        c += sums[w][2];
        any |= bits[w];
    }
    if (blockIdx.y == 0) {
        LayerScale s;
        s.t1 = 1.001f * __builtin_sqrtf(a) + kSlack;
        s.t1_max = 1.001f * __builtin_sqrtf(b) + kSlack;
        s.b1 = 1.001f * __builtin_sqrtf(c) + kSlack;
        s.no_bias = any == 0;
        *reinterpret_cast<LayerScale*>(rec) = s;
    } else {
        WordScale s;
        s.s2 = static_cast<float>(1.001 * kU) * (__builtin_sqrtf(a) + static_cast<float>(hidden) * kSlack);
        s.w2 = 1.001f * __builtin_sqrtf(b) + kSlack;
        s.zeros = any;
        s.uneven = !(s.w2 * c <= kUneven * static_cast<float>(32 - __builtin_popcount(any)));   // also where one is no number
        reinterpret_cast<WordScale*>(rec)[blockIdx.y] = s;
    }
}

// h = a / (1 + exp(-a)) with the hardware's exponential and reciprocal
__device__ __forceinline__ float fast_silu(float a)
{
    return a * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(a * -0x1.715476p+0f));
}

// The hi / lo split of bulk::split8, each h - hi in one instruction: h - 1 * hi[0] - 0 * hi[1] (exact; where hi[1] is no
// number the key is not settled).
__device__ __forceinline__ void split8(const float (&h)[8], bf16x8_t& hi, bf16x8_t& lo)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    union { bf16x8_t v; bf16x2_t p[4]; } a, b;
    // {-1, 0} and {0, -1}, in registers: as a literal of the instruction the first is taken for the second
    uint32_t minus_first = 0x0000bf80u, minus_second = 0xbf800000u;
    asm("" : "+s"(minus_first), "+s"(minus_second));
    const bf16x2_t first = __builtin_bit_cast(bf16x2_t, minus_first), second = __builtin_bit_cast(bf16x2_t, minus_second);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        a.p[p] = __builtin_convertvector(f32x2_t{h[2 * p], h[2 * p + 1]}, bf16x2_t);
        b.p[p] = __builtin_convertvector(f32x2_t{__builtin_amdgcn_fdot2_f32_bf16(a.p[p], first, h[2 * p], false),
                                                 __builtin_amdgcn_fdot2_f32_bf16(a.p[p], second, h[2 * p + 1], false)}, bf16x2_t);
    }
    hi = a.v;
    lo = b.v;
}

// What looks at the outputs of a tile and their bounds: nothing in the library; tests compare them with the chain's.
struct NoRecord {
    // a lane's 16 outputs of a word of vector `row`, from 16 half on in the order of the word's bits, and the bound of output v of them
    template <typename Bound>
    __device__ __forceinline__ void operator()(int xhead, int64_t row, int word, int half, const f32x16_t& y, Bound bound_of) const {}
};

// A wavefront takes tiles of 32 keys alone.  Layer 1 (rows = hidden units of a block of 32, columns = keys) leaves eight
// consecutive units of a key in eight accumulators of a lane, which is how layer 2 (rows = the outputs of a code word,
// columns = keys) reads them: activations stay in the registers of their wavefront.  The weights of both layers are in
// LDS as the instruction reads them, 16 bytes a lane: all of them (RESIDENT), fetched once per workgroup, or one step's at
// a time, double-buffered, for eight tiles at once.
// A step is layer 1 of a block (of the next tile's first after a tile's last), beside the activations and layer 2 of the
// block before: matrix and vector instructions that do not wait for each other.
// Lane c + 32 half has outputs 16 half .. 16 half + 15 (in bit order, highest first) of a word of key c, so a code is
// shifted together in the lane from the signs.
template <int WM, bool RESIDENT, typename Record>
__global__ __launch_bounds__(kWaves * 64, 2) void hash_screen_kernel(HashArgs a, const char* __restrict__ scales, const uint4* __restrict__ operands, int rounds, Record record)
{
    constexpr int NT = kWaves * 64, TK = bulk::kTile, OPS = operands_of(WM);
    extern __shared__ __align__(16) float lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, half = lane >> 5;
    const int xhead = blockIdx.y;
    const int whead = whead_of(a, xhead);
    const bf16_raw* b1 = static_cast<const bf16_raw*>(a.b1) + static_cast<int64_t>(whead) * a.hidden;
    const LayerScale* ls = reinterpret_cast<const LayerScale*>(scales + static_cast<int64_t>(whead) * (1 + a.W) * 16);
    const WordScale* ws = reinterpret_cast<const WordScale*>(ls) + 1;
    const int nub = blocks_of(a.hidden), W = a.W;
    const uint4* from = operands + static_cast<int64_t>(whead) * nub * OPS * 64;
    float* bias = lds;                                       // [blocks][32]
    uint4* ops = reinterpret_cast<uint4*>(bias + nub * 32);  // [blocks, or two buffers][OPS][64]

    const bf16_raw* xbase = static_cast<const bf16_raw*>(a.x) + xhead * a.x_head_stride + a.x_row0 * kHeadDim;
    const int64_t n_tiles = (a.n_rows + TK - 1) / TK, tile0 = static_cast<int64_t>(blockIdx.x) * rounds * kWaves;
    const int64_t segments = bulk::segments_of(a);
    RowScale* rows = reinterpret_cast<RowScale*>(ops + (RESIDENT ? nub : 2) * OPS * 64);   // [W][32]
    // open rows, where the second pass is shared out by them: each wavefront counts its own, the workgroup adds those of the first segments up in LDS and then to the segments' counts
    // (an addition in memory for every tile: 8 heads x 65536, 128 -> 256 -> 128, both passes, 334 us; so 235)
    uint32_t* opened = reinterpret_cast<uint32_t*>(rows + W * 32);
    const int seg0 = static_cast<int>(tile0 / (bulk::kOpenSegment / TK));
    int seg = seg0, n_opened = 0;
    if (tid < kNear) opened[tid] = 0;
    auto count_opened = [&]() {
        if (lane != 0 || n_opened == 0 || !a.open_counts) return;
        if (seg - seg0 < kNear) atomicAdd(opened + (seg - seg0), static_cast<uint32_t>(n_opened));
        else atomicAdd(a.open_counts + (xhead * segments + seg) * bulk::kCountStride, static_cast<uint32_t>(n_opened));
    };
    uint4 x[8];
    auto fetch_x = [&](int64_t tile) {
        const int64_t row = min(tile * TK + c, a.n_rows - 1);   // rows past the end: a stand-in, never stored
#pragma unroll
        for (int s = 0; s < 8; ++s) x[s] = *reinterpret_cast<const uint4*>(xbase + row * kHeadDim + (2 * s + half) * 8);
    };
    fetch_x(tile0 + wave);
    for (int i = tid; i < nub * 32; i += NT) bias[i] = i < a.hidden ? load1(b1 + i) : 0.0f;
    // operand f of a step: layer 1 of the block behind `ub`, layer 2 of `ub`
    auto bring = [&](int ub, int buf) {
        const int behind = ub + 1 < nub ? ub + 1 : 0;
#pragma unroll
        for (int p = 0; p < (OPS + kWaves - 1) / kWaves; ++p) {
            const int f = wave + p * kWaves;
            if (f < OPS)
                __builtin_amdgcn_global_load_lds(
                    reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(reinterpret_cast<uintptr_t>(from + ((f < 8 ? behind : ub) * OPS + f) * 64 + lane)),
                    reinterpret_cast<__attribute__((address_space(3))) uint32_t*>(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(ops + (buf * OPS + f) * 64))), 16, 0, 0);
        }
    };
    // what this wavefront has asked for is there (also in LDS), then everybody's
    auto arrive = [&]() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
    if constexpr (RESIDENT) {
        const bf16_raw* w1 = static_cast<const bf16_raw*>(a.w1) + static_cast<int64_t>(whead) * a.hidden * kHeadDim;
        const bf16_raw* w2 = static_cast<const bf16_raw*>(a.w2) + static_cast<int64_t>(whead) * a.L * a.hidden;
        const int n = nub * OPS;
        for (int f0 = wave; f0 < n; f0 += kWaves * 8) {
            uint4 v[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) { const int f = min(f0 + p * kWaves, n - 1); v[p] = operand(w1, w2, a.hidden, W, WM, f / OPS, f % OPS, lane); }
#pragma unroll
            for (int p = 0; p < 8; ++p) { const int f = f0 + p * kWaves; if (f < n) ops[f * 64 + lane] = v[p]; }
        }
    } else {
        bring(nub - 1, 1);   // layer 1 of block 0
        bring(0, 0);
    }
    static_assert(kWords * 32 <= NT, "one record a thread");
    uint32_t uneven = 0;
#pragma unroll
    for (int w = 0; w < WM; ++w) uneven |= ws[min(w, W - 1)].uneven;
    if (uneven && tid < W * 32) rows[tid] = row_scales(scales, a.n_wheads, whead, W)[tid];
    const float t1 = ls->t1, t1_max = ls->t1_max, bn = ls->b1;
    const bool no_bias = ls->no_bias != 0;
    arrive();

    f32x16_t y[WM], h;
    float xn, ca, aa, hh;    // ||x||; sums of squares of S_32, S_64 and S_96, of a', of h'
    bool nothing;            // the key and b1 are zeros: so is every output, and the code
    // a new tile: its norm, and outputs of 0 (rows of zeros: far from zero, and negative)
    auto start = [&]() {
        float xx = 0.0f;
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const uint32_t d[4] = {x[s].x, x[s].y, x[s].z, x[s].w};
#pragma unroll
            for (int p = 0; p < 4; ++p) xx = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, d[p]), __builtin_bit_cast(bf16x2_t, d[p]), xx, false);
        }
        xx = add_halves(xx);
        nothing = false;
        if (bulk::rare(xx == 0.0f && no_bias)) {
            uint32_t bits = 0;
#pragma unroll
            for (int s = 0; s < 8; ++s) bits |= bulk::magnitude_bits(x[s]);
            nothing = no_bias && (bits | other_half(bits)) == 0;
        }
        xn = 1.001f * __builtin_amdgcn_sqrtf(xx) + kSlack;
    };
    auto clear = [&]() {
        aa = hh = 0.0f;
#pragma unroll
        for (int w = 0; w < WM; ++w) {
#pragma unroll
            for (int v = 0; v < 16; ++v) y[w][v] = 0.0f;
            if (w < W) {
                const uint32_t z = ws[w].zeros;
                if (z) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) y[w][v] = (z >> (v + 16 * half)) & 1 ? -1e30f : 0.0f;
                }
            }
        }
    };
    // layer 1 of block ub; the sum of squares of its sums on the way
    auto layer1 = [&](int ub, const uint4* op, f32x16_t& acc) {
        float sum = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 f = *reinterpret_cast<const float4*>(bias + ub * 32 + 16 * (q / 2) + 8 * half + 4 * (q % 2));
            acc[4 * q] = f.x; acc[4 * q + 1] = f.y; acc[4 * q + 2] = f.z; acc[4 * q + 3] = f.w;
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, op[s * 64]), __builtin_bit_cast(bf16x8_t, x[s]), acc, 0, 0, 0);
            if (s == 1 || s == 3 || s == 5) {
#pragma unroll
                for (int v = 0; v < 16; ++v) sum = __builtin_fmaf(acc[v], acc[v], sum);
            }
        }
        return sum;
    };
    // the activations of a block, and its part of the outputs
    auto layer2 = [&](const uint4* op) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float h8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float av = h[8 * j + e], hv = fast_silu(av);
                aa = __builtin_fmaf(av, av, aa);
                hh = __builtin_fmaf(hv, hv, hh);
                h8[e] = hv;
            }
            bf16x8_t hi, lo;
            // (the sum first, so that the split may overwrite h8)
            asm volatile("" : "+v"(hh), "+v"(h8[0]), "+v"(h8[1]), "+v"(h8[2]), "+v"(h8[3]), "+v"(h8[4]), "+v"(h8[5]), "+v"(h8[6]), "+v"(h8[7]));
            split8(h8, hi, lo);
#pragma unroll
            for (int w = 0; w < WM; ++w) {
                const bf16x8_t b = __builtin_bit_cast(bf16x8_t, op[(8 + j * WM + w) * 64]);
                y[w] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, hi, y[w], 0, 0, 0);
                y[w] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, lo, y[w], 0, 0, 0);
            }
        }
    };
    // the tile's bound, codes and open keys
    auto finish = [&](int64_t tile) {
        ca = add_halves(ca);
        aa = add_halves(aa);
        hh = add_halves(hh);
        constexpr float u = static_cast<float>(1.02 * kU);
        const float an = 1.001f * __builtin_amdgcn_sqrtf(aa) + kSlack, hn = 1.001f * __builtin_amdgcn_sqrtf(hh) + kSlack;
        const float sums = 24.0f * bn + 76.3f * (1.001f * __builtin_amdgcn_sqrtf(ca) + kSlack) + 20.0f * an;   // 44 sqrt(3) for the three of them
        const float da = u * (t1 * xn + sums);                                                         // >= ||a - a'||
        const float slope = 0.5f * t1 + 0.5f * t1_max * (an + da), steepest = 1.1f * t1;
        const float dh = u * ((slope < steepest ? slope : steepest) * xn + 1.1f * sums + 12.0f * hn + 2.0f * an);
        auto own_bound = [&](int w, int v) { const RowScale& r = rows[w * 32 + 16 * half + v]; return 1.002f * (r.s2 * (hn + dh) + r.w2 * dh); };
        // signs, and the distance of the nearest output from zero
        uint32_t code[WM];
        bool sure = true;
#pragma unroll
        for (int w = 0; w < WM; ++w) {
            if (w >= W) continue;
            uint32_t s = 0;
            float nearest = INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                s = __builtin_amdgcn_alignbit(s, __float_as_uint(y[w][v]), 31);
                nearest = fminf(nearest, __builtin_fabsf(y[w][v]));
            }
            const float bound = 1.002f * (ws[w].s2 * (hn + dh) + ws[w].w2 * dh);
            sure = sure && nearest >= bound && bound < 1e25f;
            code[w] = ~s & 0xffffu;   // a settled output is no zero
            if (tile * TK + c < a.n_rows) record(xhead, tile * TK + c, w, half, y[w], [&](int v) { return ws[w].uneven ? own_bound(w, v) : bound; });
        }
        // each output and the bound of its own row (behind all words: a branch in each, 8 heads x 131072, 128 -> 512 -> 256, 787 us, so 762;
        // 32 x 131072, 128 -> 256 -> 128, 926 and 914)
        if (uneven && __ballot(!sure)) {
            sure = true;
#pragma unroll
            for (int w = 0; w < WM; ++w) {
                if (w >= W) continue;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float b = own_bound(w, v);
                    sure = sure && __builtin_fabsf(y[w][v]) >= b && b < 1e25f;
                    if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (registers)
                }
            }
        }
        uint32_t open = sure || nothing ? 0u : 1u;
        open |= other_half(open);
        const bool mine = half == 0 && tile * TK + c < a.n_rows;
        const uint32_t marked = static_cast<uint32_t>(__ballot(mine && open != 0));
#pragma unroll
        for (int w = 0; w < WM; ++w) {
            if (w >= W) continue;
            code[w] = (code[w] << 16) | other_half(code[w]);
            if (nothing) code[w] = 0;
        }
        if (mine) {
            uint32_t* to = a.codes + xhead * a.code_head_stride + (a.code_row0 + tile * TK + c) * W;
#pragma unroll
            for (int w = 0; w < WM; ++w)
                if (w < W) to[w] = code[w];
        }
        if (lane == 0 && tile < n_tiles) a.open[xhead * a.open_stride + tile] = marked;
        const int s = static_cast<int>(tile / (bulk::kOpenSegment / TK));
        if (s != seg) {
            count_opened();
            seg = s;
            n_opened = 0;
        }
        n_opened += __builtin_popcount(marked);
    };

    // operands of a step: layer 1 of the block behind `ub`, layer 2 of `ub`
    int buf = 0;
    auto first_ops = [&](int ub) { return ops + (RESIDENT ? (ub + 1 < nub ? ub + 1 : 0) : buf) * OPS * 64 + lane; };
    auto second_ops = [&](int ub) { return ops + (RESIDENT ? ub : buf) * OPS * 64 + lane; };
    auto next_step = [&]() {
        if constexpr (!RESIDENT) {
            arrive();
            buf ^= 1;
        }
    };
    start();
    clear();
    ca = layer1(0, RESIDENT ? ops + lane : ops + OPS * 64 + lane, h);
    if constexpr (!RESIDENT) __syncthreads();   // before step 0 brings step 1's operands over these
    for (int round = 0; round < rounds; ++round) {
        const int64_t tile = tile0 + round * kWaves + wave;
        if constexpr (RESIDENT) { if (tile >= n_tiles) break; }   // (otherwise every wavefront meets the barriers)
        f32x16_t next;
#pragma unroll 1
        for (int ub = 0; ub < nub - 2; ++ub) {
            if constexpr (!RESIDENT) bring(ub + 1, buf ^ 1);
            ca += layer1(ub + 1, first_ops(ub), next);
            layer2(second_ops(ub));
            h = next;
            next_step();
        }
        if constexpr (!RESIDENT) bring(nub - 1, buf ^ 1);
        ca += layer1(nub - 1, first_ops(nub - 2), next);
        fetch_x(min(tile + kWaves, n_tiles - 1));   // the next tile's, in flight during the rest of this step
        layer2(second_ops(nub - 2));
        h = next;
        next_step();
        if constexpr (!RESIDENT) bring(0, buf ^ 1);
        const float ca_next = layer1(0, first_ops(nub - 1), next);
        layer2(second_ops(nub - 1));
        h = next;
        finish(tile);
        start();
        clear();
        ca = ca_next;
        next_step();
    }
    if (!a.open_counts) return;
    count_opened();
    __syncthreads();
    if (tid < kNear && opened[tid] != 0) atomicAdd(a.open_counts + (xhead * segments + seg0 + tid) * bulk::kCountStride, opened[tid]);
}

inline size_t lds_bytes(int hidden, int W, bool resident)
{
    const size_t nub = blocks_of(hidden), words = words_for(W);
    return nub * 32 * sizeof(float) + (resident ? nub : 2) * operands_of(static_cast<int>(words)) * 64 * sizeof(uint4) + W * 32 * sizeof(RowScale) + kNear * sizeof(uint32_t);
}

// Whether a workgroup's LDS (160 KB) holds the operands of all blocks.
inline bool resident(int hidden, int W) { return lds_bytes(hidden, W, true) <= 160 * 1024; }

template <int WM, bool RESIDENT, typename Record>
int launch_kernel(spotlight_ctx* ctx, const HashArgs& a, const char* scales, int n_xheads, int stage, Record record)
{
    const size_t lds = lds_bytes(a.hidden, a.W, RESIDENT);
    auto kern = hash_screen_kernel<WM, RESIDENT, Record>;
    if (allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kern), lds) != SPOTLIGHT_OK) return SPOTLIGHT_ERR_HIP;
    const int64_t all_rounds = (a.n_rows + bulk::kTile * kWaves - 1) / (bulk::kTile * kWaves);
    const int rounds = bulk::rounds_of(all_rounds, n_xheads, ctx->n_cus);
    dim3 grid(static_cast<unsigned>((all_rounds + rounds - 1) / rounds), static_cast<unsigned>(n_xheads));
    StageTimer timer(ctx, stage, true);
    timer.launch(kern, grid, dim3(kWaves * 64), lds, a, scales, static_cast<const uint4*>(a.operands), rounds, record);
    return hip_rc(hipGetLastError());
}

template <int WM, typename Record>
int launch_words(spotlight_ctx* ctx, const HashArgs& a, const char* scales, int n_xheads, int stage, Record record)
{
    if (resident(a.hidden, a.W)) return launch_kernel<WM, true>(ctx, a, scales, n_xheads, stage, record);
    return launch_kernel<WM, false>(ctx, a, scales, n_xheads, stage, record);
}

// Networks that the kernels of both passes take.
inline bool serves(int hidden, int W) { return hidden > 0 && hidden % 16 == 0 && hidden <= 1024 && W <= kWords; }

// Whether two passes serve this job (bfloat16 vectors and weights): a network that the kernels of the second one take,
// and enough tiles, since a workgroup of each pass fetches the weights and a tile of open rows is hashed by few wavefronts
// of the chip.  One pass against two, 8 and 64 heads, 32768, 65536 and 131072 vectors in all: 64 -> 32 21, 39, 63 and 28, 31,
// 35 us; 256 -> 128 48, 80, 148 and 60, 68, 83; 256 -> 256 62, 109, 201 and 84, 87, 135; 512 -> 256 127, 224, 431 and 128,
// 153, 243; 1024 -> 256 311, 594, 1156 and 288, 438, 800.  Heads of 128 vectors fill half a round: 512 of them, 256 -> 256
// 108 against 132 us.
inline bool applies(const spotlight_ctx* ctx, const HashArgs& a, int n_xheads)
{
    if (!a.open || !a.wnorm || !serves(a.hidden, a.W) || ctx->max_lds < 160 * 1024) return false;
    const int64_t tiles = (a.n_rows + bulk::kTile - 1) / bulk::kTile * n_xheads;
    if (a.n_rows < bulk::kTile * kWaves || tiles < 8 * static_cast<int64_t>(ctx->n_cus)) return false;
    if (a.W <= 4 || resident(a.hidden, a.W)) return true;
    // Codes of more than 128 bits whose weights do not fit into LDS gain least, so they need rounds of the first pass that are filled: by the heads, and by
    // the tiles of a head.  256 -> 256, one pass and two: 300 heads x 257 174 and 240 us, 257 x 288 164 and 227, 256 x 300 145 and 162, 300 x 384 228 and
    // 252; 200 x 352 152 and 137, 257 x 511 269 and 244.  512 -> 256: 300 x 257 377 and 433, 257 x 288 354 and 482; 300 x 384 492 and 473, 228 x 257 311 and 264.
    const int64_t all_rounds = (a.n_rows + bulk::kTile * kWaves - 1) / (bulk::kTile * kWaves);
    const int rounds = bulk::rounds_of(all_rounds, n_xheads, ctx->n_cus);
    const int64_t groups = (all_rounds + rounds - 1) / rounds * n_xheads;
    const int64_t room = (groups + ctx->n_cus - 1) / ctx->n_cus * rounds * ctx->n_cus * kWaves;   // tiles there would be time for
    if (a.hidden > 256) return 20 * tiles >= 7 * room;
    return 2 * tiles >= room && 3 * tiles >= 2 * all_rounds * kWaves * n_xheads;
}

template <typename Record = NoRecord>
int launch(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage, Record record = {})
{
    char* scales = static_cast<char*>(a.scales);
    const int n_operands = resident(a.hidden, a.W) ? 0 : blocks_of(a.hidden) * operands_of(words_for(a.W));
    StageTimer timer(ctx, stage, true);
    timer.launch(scales_kernel<8>, dim3(static_cast<unsigned>(a.n_wheads), static_cast<unsigned>(1 + a.W + (n_operands + kPerBlock - 1) / kPerBlock)), dim3(kThreads), 0,
                 static_cast<const bf16_raw*>(a.w1), static_cast<const bf16_raw*>(a.b1), static_cast<const bf16_raw*>(a.w2), scales,
                 static_cast<uint4*>(a.operands), a.open_counts, a.open_counts ? static_cast<int>(bulk::segments_of(a) * n_xheads) : 0, a.hidden, a.L);
    if (hipGetLastError() != hipSuccess) return SPOTLIGHT_ERR_HIP;
    if (a.W <= 2) return launch_words<2>(ctx, a, scales, n_xheads, stage, record);
    if (a.W <= 4) return launch_words<4>(ctx, a, scales, n_xheads, stage, record);
    return launch_words<8>(ctx, a, scales, n_xheads, stage, record);
}

}  // namespace screen
}  // namespace spotlight
