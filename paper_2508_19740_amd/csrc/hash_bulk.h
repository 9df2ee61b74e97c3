// Bulk hashing on the matrix cores (paper Sec. 3.2 Eq. 4-6): the code cache built after a prefill.
//
// The codes are defined by one binary32 chain per output (increasing index, one fused multiply-add
// per term).  v_mfma_f32_32x32x2_f32 computes exactly that: an instruction adds the products of
// two consecutive k to each of 32 x 32 accumulators, first the even k (lanes 0-31 of the operands),
// then the odd k (lanes 32-63), each as one correctly rounded fused multiply-add with denormals
// kept.  A sequence of these instructions is therefore the defined chain, bit for bit, at twice the
// rate of the vector ALU's unpacked fused multiply-add (153 against 78.6 TFLOP/s measured / peak).
// (tests/test_gpu_bulk_hash.py holds the builtin to the chain: wide exponents, denormal products,
// overflow.)  Unlike the bfloat16 matrix instructions, which run beside the vector ALU, it does NOT
// overlap with it: vector and binary32 matrix instructions of two wavefronts of one SIMD took the sum
// of their times (481 + 306 -> 783 us; bfloat16: 518 + 301 -> 535 us).  So these kernels are bound by
// matrix cycles PLUS vector cycles, and every vector instruction per output counts.
//
// A workgroup of NW wavefronts hashes a run of tiles of 32 vectors of one head.
//
// Layer 1 (rows = hidden units, columns = vectors): a wavefront owns blocks of 32 hidden units; its
//   weights stay in registers for the whole run of tiles, so they are read once per run (they are
//   a row per lane in memory: every load touches 32 cache lines, and re-reading them for every tile
//   would keep the texture-address unit busier than the matrix cores).  The x tile sits in LDS as
//   [k][vector], so the operand of a step is one conflict-free 4-byte LDS read.
// Layer 2, exact (rows = vectors, columns = the 32 outputs of ONE code word in bit order, so that a
//   ballot over an accumulator register is two packed words): the same instruction over the hidden
//   activations, [unit][vector] in LDS.  Binary32 weights, 1024-bit codes, hidden widths that are no
//   multiple of 16 or too large for the rest.
// Layer 2, certified (bfloat16 weights): only the SIGN of an output is needed, so it runs on
//   v_mfma_f32_32x32x16_bf16, 16 times the rate.  Each activation is split into hi + lo (both
//   bfloat16, |h - hi - lo| <= 2^-17 |h|), so the products are exact and two accumulating passes give
//   y to within
//     |y_mfma - y_chain| <= eps * sum_i |W2[j][i] h_i| <= eps * ||W2[j]|| * ||h||
//   with eps = 1.01 * 2^-24 * (0.875 * hidden + 23 + 128).  Both round partial sums S_k, the chain each by at most 2^-24 |S_k|,
//   the matrix core every eighth of hi and of lo by at most three times that (and 2^-24 * 10 times the largest product of
//   the eight: tests/test_gpu_hash_screen.py holds the instruction to it).  In the first half S_k is at most the terms so
//   far, in the second at most y and the terms to come: every term counts for hidden / 2 sums of the chain and
//   hidden / 8 of the matrix core at most (y's part is far inside the factor of 1.01).
//   Norms below 1e-12 count as infinite: the bound is then never below 1e-29, and what a conversion or the
//   matrix core flushes (1.2e-38 a term) is far inside its factor of 1.01.  The sign of
//   y_mfma is the chain's wherever |y_mfma| reaches that bound; the few outputs that do not
//   (0.02 - 0.15 %) are recomputed with the chain from the binary32 activations still in LDS.
//   While every addition was taken to err by a unit in its last place, eps was 4.5 to 5.5 times this.
#pragma once
#include <algorithm>

#include "hash_vec.h"

namespace spotlight {
namespace bulk {
using namespace hashdev;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kTile = 32;       // vectors per tile
// A norm from its square, for the bound: where the square is so small that its terms may underflow, no bound
// (infinity: nothing is settled).  Finite norms of both sides also keep every partial sum finite.
//
// A vector of zeros (padding in front of a prompt) has y = 0 exactly, or NaN beside a weight that is no number:
// bit 0 either way, nothing to recompute.  So has an output row of zeros (a code filled up to whole words).  The
// square is 0 exactly where all elements are zeros (kTinySquare stands for one that underflowed): norm and
// bound are then 0, and y = 0 is settled.  Keys of zeros, with all their outputs sent to the chain and settled:
// 512 heads x 313, linear, 512 bits, 4991 and 78 us; 64 heads x 30, 128 -> 512 -> 256, 222 and 39 us.
constexpr float kTinySquare = 1e-37f;
__device__ __forceinline__ float square_of(float s, uint32_t bits) { return s == 0.0f && bits != 0 ? kTinySquare : s; }   // bits: of the elements
__device__ __forceinline__ float norm_of(float s) { return s < 1e-24f ? (s == 0.0f ? 0.0f : INFINITY) : __builtin_sqrtf(s); }
// false where either side is NaN, or one norm is infinite and the other 0
__device__ __forceinline__ bool settled(float y, float tcol, float hn) { return __builtin_fabsf(y) >= tcol * hn; }
__device__ __forceinline__ uint32_t magnitude_bits(const uint4& bf16x8) { return (bf16x8.x | bf16x8.y | bf16x8.z | bf16x8.w) & 0x7fff7fffu; }
__device__ __forceinline__ uint32_t magnitude_bits(const float4& f)
{
    return (__float_as_uint(f.x) | __float_as_uint(f.y) | __float_as_uint(f.z) | __float_as_uint(f.w)) & 0x7fffffffu;
}
__device__ __forceinline__ uint32_t magnitude_bits(const Raw8<bf16_raw>& r) { return magnitude_bits(r.u); }
__device__ __forceinline__ uint32_t magnitude_bits(const Raw8<float>& r) { return magnitude_bits(r.a) | magnitude_bits(r.b); }
__device__ __forceinline__ uint32_t magnitude_bits(const bf16_raw* row, int n)   // of n weights in memory
{
    uint32_t bits = 0;
#pragma unroll 1
    for (int i = 0; i < n; i += 8) bits |= magnitude_bits(*reinterpret_cast<const uint4*>(row + i));
    return bits;
}
// whether a lane has the condition; what follows is seldom run and kept out of the way
__device__ __forceinline__ bool rare(bool condition) { return __builtin_expect(__ballot(condition) != 0, 0); }

constexpr int kListCap = 1024;  // outputs of a tile that may go to the recomputation

struct Scratch {   // lives in the x tile's LDS once layer 1 is done with it
    float part[16][kTile];
    float hn[kTile];              // ||h_t||
    uint32_t codes[kTile][16];
    uint16_t list[kListCap];
    uint32_t count;
};
static_assert(sizeof(Scratch) <= sizeof(float) * kHeadDim / 2 * kTile, "fits in the x tile");

// hi / lo split of 8 activations into two MFMA operands: hi = bf16(h) and lo = bf16(h - hi), both
// rounded to nearest by the packed conversion instruction; h - hi is exact.
__device__ __forceinline__ void split8(const float (&h)[8], bf16x8_t& hi, bf16x8_t& lo)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    union { bf16x8_t v; uint32_t u[4]; } a, b;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const f32x2_t hv = {h[2 * p], h[2 * p + 1]};
        const uint32_t hp = __builtin_bit_cast(uint32_t, __builtin_convertvector(hv, bf16x2_t));
        const f32x2_t rv = {h[2 * p] - __uint_as_float(hp << 16), h[2 * p + 1] - __uint_as_float(hp & 0xffff0000u)};
        a.u[p] = hp;
        b.u[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rv, bf16x2_t));
    }
    hi = a.v;
    lo = b.v;
}

// the hi part of the split alone
__device__ __forceinline__ uint4 round8(const float4& f0, const float4& f1)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const auto two = [](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{x, y}, bf16x2_t)); };
    return make_uint4(two(f0.x, f0.y), two(f0.z, f0.w), two(f1.x, f1.y), two(f1.z, f1.w));
}

// Sum over the 16 lanes of a row, in every lane: rotations, no LDS.
__device__ __forceinline__ float add_across_16(float x)
{
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, true));  // row_ror:8
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, true));  // row_ror:4
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xf, 0xf, true));  // row_ror:2
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xf, 0xf, true));  // row_ror:1
    return x;
}

// 4 consecutive weights in their stored form
template <typename WT> struct Raw4;
template <> struct Raw4<float> { float4 v; };
template <> struct Raw4<bf16_raw> { uint2 v; };
__device__ __forceinline__ void load_raw(const float* p, Raw4<float>& r) { r.v = *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ void load_raw(const bf16_raw* p, Raw4<bf16_raw>& r) { r.v = *reinterpret_cast<const uint2*>(p); }
__device__ __forceinline__ void expand(const Raw4<float>& r, float (&o)[4]) { o[0] = r.v.x; o[1] = r.v.y; o[2] = r.v.z; o[3] = r.v.w; }
__device__ __forceinline__ void expand(const Raw4<bf16_raw>& r, float (&o)[4])
{
    o[0] = __uint_as_float(r.v.x << 16); o[1] = __uint_as_float(r.v.x & 0xffff0000u);
    o[2] = __uint_as_float(r.v.y << 16); o[3] = __uint_as_float(r.v.y & 0xffff0000u);
}

// 4 consecutive biases, one element at a time: b1 may start at any element (a slice of one flat parameter
// buffer), where the calls ask W1 and W2 for 16 bytes.
template <typename WT> __host__ __device__ inline void load_bias4(const WT* p, float (&o)[4])
{
    for (int e = 0; e < 4; ++e) o[e] = load1(p + e);
}

// Turns 8 consecutive weights of a row, 4 in each half of the wavefront (lower half: k .. k+3, upper
// half: k+4 .. k+7), into the operands of four consecutive steps (lower half: even k, upper: odd k).
__device__ __forceinline__ void to_steps(float (&v)[4])
{
    float s[4];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        // exchanges the upper half of the first with the lower half of the second
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2 * p]), __float_as_uint(v[2 * p + 1]), false, false);
        s[p] = __uint_as_float(r[0]);
        s[p + 2] = __uint_as_float(r[1]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = s[e];
}

// One lane's operands of the 64 steps of layer 1 for one block of 32 hidden units: bfloat16 weights
// two steps to a register, binary32 weights one.
template <typename WT> struct UnitBlock;
template <> struct UnitBlock<bf16_raw> {
    uint32_t w[32];
    __device__ __forceinline__ void put(int g, const float (&v)[4])
    {
        w[2 * g] = (__float_as_uint(v[0]) >> 16) | __float_as_uint(v[1]);
        w[2 * g + 1] = (__float_as_uint(v[2]) >> 16) | __float_as_uint(v[3]);
    }
    __device__ __forceinline__ float step(int s) const { return __uint_as_float((s & 1) ? w[s >> 1] & 0xffff0000u : w[s >> 1] << 16); }
    // keeps the compiler from unpacking all steps once, in front of the loop over the tiles, into twice the registers
    __device__ __forceinline__ void stay_packed()
    {
#pragma unroll
        for (int i = 0; i < 32; ++i) asm volatile("" : "+v"(w[i]));
    }
};
template <> struct UnitBlock<float> {
    float w[64];
    __device__ __forceinline__ void put(int g, const float (&v)[4])
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[4 * g + e] = v[e];
    }
    __device__ __forceinline__ float step(int s) const { return w[s]; }
    __device__ __forceinline__ void stay_packed() {}
};

// The x tile in LDS, [step][vector]: bfloat16 vectors with both k of a step in one word (half the
// room, so that one more workgroup fits a compute unit), binary32 vectors a word for each k.
template <typename XT> struct XTile;
template <> struct XTile<bf16_raw> {
    static constexpr int kFloats = kHeadDim / 2 * kTile;
    // elements 8 k8 .. 8 k8 + 7 of vector t
    static __device__ __forceinline__ void put(float* xs, int k8, int t, const Raw8<bf16_raw>& r)
    {
        const uint32_t v[4] = {r.u.x, r.u.y, r.u.z, r.u.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) reinterpret_cast<uint32_t*>(xs)[(k8 * 4 + j) * kTile + t] = v[j];
    }
    // the lane's operand of step s: the even k in the lower half of the wavefront, the odd k in the upper
    static __device__ __forceinline__ float step(const float* xs, int s, int lane)
    {
        const uint32_t v = reinterpret_cast<const uint32_t*>(xs)[s * kTile + (lane & 31)];
        return __uint_as_float(__builtin_amdgcn_perm(v, v, lane < 32 ? 0x01000c0cu : 0x03020c0cu));
    }
};
template <> struct XTile<float> {
    static constexpr int kFloats = kHeadDim * kTile;
    static __device__ __forceinline__ void put(float* xs, int k8, int t, const Raw8<float>& r)
    {
        float v[8];
        expand(r, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) xs[(k8 * 8 + j) * kTile + t] = v[j];
    }
    static __device__ __forceinline__ float step(const float* xs, int s, int lane) { return xs[s * 64 + lane]; }
};

// ||W2[j]|| of every output row of every weight head, for the bound above: 16 lanes per row.
template <int LPR>
__global__ __launch_bounds__(kThreads) void row_norm_kernel(const bf16_raw* __restrict__ w2, float* __restrict__ wnorm, int n_rows, int n)
{
    const int j = (blockIdx.x * kThreads + threadIdx.x) / LPR, sub = threadIdx.x % LPR;
    if (j >= n_rows) return;   // whole groups of LPR lanes
    float s = 0.0f;
    uint32_t bits = 0;
    for (int g = sub; g < n / 8; g += LPR) {
        Raw8<bf16_raw> raw;
        load_raw(w2 + static_cast<int64_t>(j) * n + g * 8, raw);
        float wv[8];
        expand(raw, wv);
        bits |= magnitude_bits(raw);
#pragma unroll
        for (int e = 0; e < 8; ++e) s = __builtin_fmaf(wv[e], wv[e], s);
    }
    s = square_of(s, bits);
#pragma unroll
    for (int off = 1; off < LPR; off <<= 1) s += __shfl_xor(s, off);
    if (sub == 0) wnorm[j] = norm_of(s);
}

__host__ __device__ constexpr int hidden_padded(int hidden) { return (hidden + 31) / 32 * 32; }

// The tiles of workgroup `id`, `parts` of them for every head: `longer` of a head's have run + 1 tiles, the others run (the
// last what is left).  The longer ones come first, so that a compute unit that takes several workgroups gets one of
// each kind before it gets a second longer one.
struct Share {
    int head;
    int64_t tile;
    int tiles;
};
__host__ __device__ inline Share share_of(unsigned id, unsigned parts, unsigned heads, int run, int longer)
{
    const unsigned long_ones = static_cast<unsigned>(longer) * heads;
    if (id < long_ones) return {static_cast<int>(id / longer), static_cast<int64_t>(id % longer) * (run + 1), run + 1};
    const unsigned rest = id - long_ones, others = parts - longer;
    return {static_cast<int>(rest / others), static_cast<int64_t>(longer) * (run + 1) + static_cast<int64_t>(rest % others) * run, run};
}

// The rows that a first pass left open (hash_screen.h), compacted a span at a time, so that the kernels below hash
// tiles of 32 of those alone: what does not fill a tile waits for the next span.  A segment of a head's rows is shared out
// over several workgroups, the same number of tiles of open rows each, as far as they divide: every one of them counts the
// segment's rows first, a few words a thread.  (A range of rows for each, two for every slot of the chip, had a
// tile that was not full in every range and waited for the ranges with the most: 32 heads x 131072, 128 -> 256 -> 128, 9 % open,
// 557 us; this way 527.)
constexpr int kOpenSegment = 65536;   // rows: offsets in 16 bits
constexpr int kCountStride = 32;      // words between the counts of two segments: a cache line each
constexpr int kOpenSpan = 2048;       // rows: a word of the bitmap for each lane of a wavefront
struct OpenRows {
    uint16_t row[kOpenSpan + kTile];  // in the segment
    int count, left, tiles;           // rows in the list, rows of the share not in the list yet, whole tiles of the list
    int sums[16];
    int job[4];                       // what the workgroup has: OpenJob, its segment for the tile
};

// Tiles of open rows a workgroup takes, the fewest with which `slots` of them have all `total` of the `segments` (fewer than slots);
// parts_with(q): workgroups it takes with q tiles each.
template <typename F>
__host__ __device__ inline int open_quota(int total, int segments, int slots, F parts_with)
{
    int lo = (total + slots - 1) / slots, hi = (total - 1) / (slots - segments) + 1;   // segments' remainders: at most one each
    while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (parts_with(mid) <= slots) hi = mid; else lo = mid + 1;
    }
    return hi;
}

// Workgroups of a segment, where `all` would do with q tiles each: the others of the chip's `slots` are spread over the segments, as far as each has a tile
// (28 heads x 4703, 128 -> 64 -> 64, 370 tiles for 768 workgroups: second pass 20.0 us where some have none, 14.6; 64 x 1024, 128 -> 256 -> 128, 38 and 31).
__host__ __device__ inline uint32_t open_workgroups(uint32_t tiles, uint32_t q, uint32_t all, uint32_t slots)
{
    const uint32_t spread = (tiles + q - 1) / q * slots / all;
    return spread < tiles ? spread : tiles;
}

__host__ __device__ inline int64_t segments_of(const HashArgs& a) { return (a.n_rows + kOpenSegment - 1) / kOpenSegment; }

// What a workgroup of the second pass has: share `part` of `parts` of a segment's open rows (parts 0: nothing).
struct OpenJob {
    int xhead, part, parts;
    int64_t first;                    // the segment's first tile
};
constexpr int kOpenBalanced = 256;    // segments that a wavefront shares out; with more, or few slots for each, none runs on for long

// Whether the first pass counts them and the second shares them out.  Counts take 3 to 5 us; small calls of narrow layers are over before an uneven share
// costs that.  Without and with: 100 heads x 700, 128 -> 64 -> 32 29.5 and 31.6 us, 40 x 1800, 128 -> 16 -> 32 27 and 31; 64 x 1024, 128 -> 256 -> 128 65.5 and 61.5,
// one head open for all keys 215 and 91; 8 x 8192, 128 -> 128 -> 64 35.7 and 34.9; 28 x 4703, 128 -> 64 -> 64 38.2 and 37.4, one head 160 and 48.
inline bool counts_open_rows(const HashArgs& a, int n_xheads, int n_cus)
{
    const int64_t tiles = (a.n_rows + kTile - 1) / kTile * n_xheads;
    return segments_of(a) * n_xheads <= kOpenBalanced && tiles * a.hidden > 800 * static_cast<int64_t>(n_cus);
}

// Of `n` segments, `per_head` of every head, the one that workgroup blockIdx.x of gridDim.x has, and its share there.
__device__ __forceinline__ void share_segments(OpenRows& list, const uint32_t* counts, int n, int per_head, int lane)
{
    constexpr int PL = kOpenBalanced / 64;
    uint32_t tiles[PL], total = 0;
#pragma unroll
    for (int k = 0; k < PL; ++k) {
        const int s = k * 64 + lane;
        tiles[k] = s < n ? (counts[s * kCountStride] + kTile - 1) / kTile : 0u;
        total += tiles[k];
    }
    total = wave_sum(total);
    if (lane < 4) list.job[lane] = 0;
    if (total == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    auto parts_with = [&](int q) {
        uint32_t parts = 0;
#pragma unroll
        for (int k = 0; k < PL; ++k)
            if (k * 64 < n) parts += (tiles[k] + q - 1) / static_cast<uint32_t>(q);
        return static_cast<int>(wave_sum(parts));
    };
    const uint32_t q = open_quota(static_cast<int>(total), n, static_cast<int>(gridDim.x), parts_with);
    const uint32_t all = static_cast<uint32_t>(parts_with(static_cast<int>(q)));
    uint32_t id = blockIdx.x;
#pragma unroll
    for (int k = 0; k < PL; ++k) {
        const uint32_t parts = open_workgroups(tiles[k], q, all, gridDim.x), upto = wave_inclusive_scan(parts);
        const bool here = upto - parts <= id && id < upto;
        if (here) {   // one lane at most
            const int s = k * 64 + lane;
            list.job[0] = s / per_head;
            list.job[1] = static_cast<int>(id - (upto - parts));
            list.job[2] = static_cast<int>(parts);
            list.job[3] = s % per_head;
        }
        const uint32_t before = __builtin_amdgcn_readlane(static_cast<int>(upto), 63);
        if (id < before) return;
        id -= before;
    }
}

// run > 0: that many workgroups for every segment.  run < 0: the workgroups are shared out over the segments of -run heads by the rows that
// the first pass counted there, so that a head with more of them does not run on when the others are done (8 heads x 65536, 128 -> 256 -> 128,
// one output of one head open for all keys: 1475 us with as many for each, 488 us so; equal heads 227 and 235).  Every thread of the workgroup calls it.
__device__ __forceinline__ OpenJob open_job(OpenRows& list, const HashArgs& a, int run, int wave, int lane)
{
    if (run > 0) return {static_cast<int>(blockIdx.y), static_cast<int>(blockIdx.x % run), run, static_cast<int64_t>(blockIdx.x / run) * (kOpenSegment / kTile)};
    const int per_head = static_cast<int>(segments_of(a));
    if (wave == 0) share_segments(list, a.open_counts, -run * per_head, per_head, lane);
    __syncthreads();
    const auto of = [&](int i) { return __builtin_amdgcn_readfirstlane(list.job[i]); };
    return {of(0), of(1), of(2), static_cast<int64_t>(of(3)) * (kOpenSegment / kTile)};
}

// The open rows of a segment that belong to a share, counted in the order of the rows.
struct OpenShare { int from, to; };
__host__ __device__ inline OpenShare open_share(int total, int part, int parts)
{
    const int all = (total + kTile - 1) / kTile;
    const int from = static_cast<int>(static_cast<int64_t>(all) * part / parts) * kTile, to = static_cast<int>(static_cast<int64_t>(all) * (part + 1) / parts) * kTile;
    return {from, to < total ? to : total};
}

// A word of the bitmap without what lies behind the segment's last row.
__host__ __device__ inline uint32_t open_word(const uint32_t* open, int word, int n_rows)
{
    const int rows = n_rows - word * 32;
    return rows <= 0 ? 0u : rows >= 32 ? open[word] : open[word] & ((1u << rows) - 1u);
}

// Puts a word's open rows into the list, the first at `at` behind the `rest` rows there; rows of the shares before have at < 0.
__host__ __device__ inline void list_rows(uint16_t* list, uint32_t bits, int word, int rest, int at, int left)
{
    for (; bits != 0; bits &= bits - 1, ++at)
        if (at >= 0 && at < left) list[rest + at] = static_cast<uint16_t>(word * 32 + __builtin_ctz(bits));
}

// Rows in the list and rows to come behind a span that ends at word `next` and had `found` rows of the share; whole tiles to hash
// now.  Behind the last word nothing comes, whatever was counted in the beginning: the walk ends also where the bitmap has changed since (another
// stream's call on the same context; its codes are undefined then, but it must not hang).
struct OpenSpan { int count, left, tiles; };
__host__ __device__ inline OpenSpan after_span(int rest, int found, int left, int next, int n_rows)
{
    const int added = found < 0 ? 0 : found < left ? found : left;
    const int to_come = next * 32 < n_rows ? left - added : 0;
    return {rest + added, to_come, to_come > 0 ? (rest + added) / kTile : (rest + added + kTile - 1) / kTile};
}

struct OpenWalk {
    OpenRows& list;
    const uint32_t* open;             // the segment's words of the bitmap
    int n_rows, next, skip;           // rows of the segment, the next word to be looked at, open rows there that belong to the shares before
    int count, left, tiles;           // as above; whole tiles of the list to be hashed now

    // Finds the share; false: it is empty.  Every thread of the workgroup calls it.
    __device__ __forceinline__ bool begin(int part, int parts, int tid, int n_threads)
    {
        const int lane = tid & 63, wave = tid >> 6, n_words = (n_rows + 31) / 32, per = (n_words + n_threads - 1) / n_threads;   // 64 words at most
        uint32_t mine = 0;
        for (int i = 0; i < per; ++i) mine += static_cast<uint32_t>(__builtin_popcount(open_word(open, tid * per + i, n_rows)));
        const int upto = static_cast<int>(wave_inclusive_scan(mine));
        if (lane == 63) list.sums[wave] = upto;
        __syncthreads();
        int before = upto - static_cast<int>(mine), total = 0;
        for (int w = 0; w < n_threads / 64; ++w) {
            before += w < wave ? list.sums[w] : 0;
            total += list.sums[w];
        }
        const OpenShare share = open_share(total, part, parts);
        if (share.from >= share.to) return false;
        if (before <= share.from && share.from < before + static_cast<int>(mine)) {
            list.count = tid * per;
            list.left = share.from - before;
        }
        __syncthreads();
        next = __builtin_amdgcn_readfirstlane(list.count);
        skip = __builtin_amdgcn_readfirstlane(list.left);
        count = tiles = 0;
        left = __builtin_amdgcn_readfirstlane(share.to - share.from);
        return true;
    }
    // Fills the list up to the next tiles; false: there are none left.  Every thread of the workgroup calls it.
    __device__ __forceinline__ bool advance(int wave, int lane)
    {
        if (left == 0) return false;
        do {
            __syncthreads();   // the tiles before are done with the list
            if (wave == 0) {
                const int rest = count - tiles * kTile;   // fewer than a tile
                const uint16_t r = list.row[tiles * kTile + min(lane, kTile - 1)];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (lane < rest) list.row[lane] = r;
                const uint32_t bits = open_word(open, next + lane, n_rows);
                const int mine = __builtin_popcount(bits), upto = static_cast<int>(wave_inclusive_scan(static_cast<uint32_t>(mine)));
                list_rows(list.row, bits, next + lane, rest, upto - mine - skip, left);
                if (lane == 63) {
                    const OpenSpan s = after_span(rest, upto - skip, left, next + kOpenSpan / 32, n_rows);
                    list.count = s.count;
                    list.left = s.left;
                    list.tiles = s.tiles;
                }
            }
            __syncthreads();
            count = __builtin_amdgcn_readfirstlane(list.count);
            left = __builtin_amdgcn_readfirstlane(list.left);
            tiles = __builtin_amdgcn_readfirstlane(list.tiles);
            next += kOpenSpan / 32;
            skip = 0;
        } while (tiles == 0 && left > 0);
        return tiles > 0;
    }
};

// Outputs of a word that a first pass settled and the chain contradicts.
__device__ __forceinline__ uint32_t settled_wrong(const HashArgs& a, int xhead, int64_t row, uint32_t before, uint32_t now)
{
    if (!a.open || (a.open[xhead * a.open_stride + row / 32] >> (row % 32)) & 1u) return 0;
    return static_cast<uint32_t>(__builtin_popcount(before ^ now));
}

// Wavefronts per SIMD the register allocation must leave room for.  8 heads x 131072 vectors, 128 -> 512 ->
// 256: four (128 registers and 38 spilled; 51 with binary32 vectors) 3.32 ms, three 3.83 ms.
constexpr int min_waves(int NW, int NBW) { return NBW == 1 && NW >= 8 ? 4 : 2; }

// NW:    wavefronts per workgroup.
// NUB:   blocks of 32 hidden units a wavefront owns, their weights in registers; 0: the linear hash;
//        -1: any number, weights read again for every tile.
// NBW:   code words per wavefront of the certified second layer; 0: exact second layer.
// AUDIT: every output of the certified second layer is also evaluated with the chain and compared
//        (distance in units of ||W2[j]|| ||h||, settled signs that disagree); totals go to a.audit.
// OPEN:  only the rows a first pass left open, of the workgroup's range of tiles.
template <typename XT, typename WT, int NW, int NUB, int NBW, bool AUDIT, bool OPEN = false>
__global__ __launch_bounds__(NW * 64, min_waves(NW, NBW)) void hash_bulk_kernel(HashArgs a, float eps, int run, int extra)
{
    constexpr int TK = kTile, NT = NW * 64;
    constexpr bool CERT = NBW > 0;
    extern __shared__ __align__(16) float lds[];
    float* xs = lds;                                   // the x tile, later Scratch
    float* hs = lds + XTile<XT>::kFloats;              // [hidden, padded to 32][TK]
    Scratch& m = *reinterpret_cast<Scratch*>(xs);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31, half = lane >> 5;
    Share share{static_cast<int>(blockIdx.y), static_cast<int64_t>(blockIdx.x) * run, run};
    if (!OPEN && extra != 0) share = share_of(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x, gridDim.y, run, extra);
    OpenJob job{};   // OPEN: in place of the share; its list is `extra` bytes into LDS
    if constexpr (OPEN) {
        job = open_job(*reinterpret_cast<OpenRows*>(reinterpret_cast<char*>(lds) + extra), a, run, wave, lane);
        if (job.parts == 0) return;
    }
    const int xhead = OPEN ? job.xhead : share.head;
    const int whead = whead_of(a, xhead);
    const WT* w1 = static_cast<const WT*>(a.w1) + static_cast<int64_t>(whead) * (a.hidden > 0 ? a.hidden : a.L) * kHeadDim;
    const WT* b1 = static_cast<const WT*>(a.b1) + static_cast<int64_t>(whead) * a.hidden;
    const int K2 = NUB == 0 ? kHeadDim : a.hidden;     // what layer 2 contracts over
    const WT* w2 = NUB == 0 ? w1 : static_cast<const WT*>(a.w2) + static_cast<int64_t>(whead) * a.L * a.hidden;
    const int nub = hidden_padded(a.hidden) / 32;

    const int64_t n_tiles = (a.n_rows + TK - 1) / TK;
    const int64_t first = OPEN ? job.first : share.tile;
    int64_t tile0 = first, tile1 = min(n_tiles, first + (OPEN ? kOpenSegment / TK : share.tiles));
    OpenWalk walk{*reinterpret_cast<OpenRows*>(reinterpret_cast<char*>(lds) + (OPEN ? extra : 0)), OPEN ? a.open + xhead * a.open_stride + first : nullptr,
                  static_cast<int>(min(a.n_rows - first * TK, static_cast<int64_t>(kOpenSegment))), 0, 0, 0, 0, 0};
    if constexpr (OPEN) {
        if (!walk.begin(job.part, job.parts, tid, NT) || !walk.advance(wave, lane)) return;
        tile0 = 0;
        tile1 = walk.tiles;
    }
    auto n_items = [&]() { return OPEN ? static_cast<int64_t>(walk.count) : a.n_rows; };
    auto row_of = [&](int64_t item) { return OPEN ? first * TK + walk.list.row[item] : item; };

    uint32_t au_outputs = 0, au_listed = 0, au_wrong = 0;   // this lane's audit totals
    float au_ratio = 0.0f;

    // Weights and biases of a block of hidden units; units past the end have zeros, i.e. activation 0.
    auto load_block = [&](int ub, UnitBlock<WT>& u) {
        const int unit = ub * 32 + c;
        const WT* row = w1 + static_cast<int64_t>(min(unit, a.hidden - 1)) * kHeadDim + 4 * half;
        Raw4<WT> raw[16];
#pragma unroll
        for (int g = 0; g < 16; ++g) load_raw(row + 8 * g, raw[g]);
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            float v[4];
            expand(raw[g], v);
            if (unit >= a.hidden) v[0] = v[1] = v[2] = v[3] = 0.0f;
            to_steps(v);
            u.put(g, v);
        }
    };
    // accumulator register v of a block holds hidden unit 8 (v / 4) + 4 half + v % 4 of it
    auto load_bias = [&](int ub, f32x16_t& acc) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int unit = ub * 32 + 8 * q + 4 * half;   // hidden is a multiple of 8: a group of four is whole
            float v[4];
            load_bias4(b1 + min(unit, a.hidden - 4), v);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * q + e] = unit < a.hidden ? v[e] : 0.0f;
        }
    };
    float sumsq;
    auto layer1 = [&](int ub, const UnitBlock<WT>& u) {
        f32x16_t acc;
        load_bias(ub, acc);
#pragma unroll
        for (int s = 0; s < kHeadDim / 2; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(u.step(s), XTile<XT>::step(xs, s, lane), acc, 0, 0, 0);
        float* h = hs + (ub * 32 + 4 * half) * TK + c;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float hv = silu(acc[v]);
            h[(8 * (v / 4) + v % 4) * TK] = hv;
            if constexpr (CERT) sumsq = __builtin_fmaf(hv, hv, sumsq);
            if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // four at a time: sixteen side by side would spill
        }
    };
    UnitBlock<WT> ublk[NUB > 0 ? NUB : 1];
    if constexpr (NUB > 0) {
#pragma unroll
        for (int i = 0; i < NUB; ++i)
            if (wave + NW * i < nub) load_block(wave + NW * i, ublk[i]);
    }

    // the x tile of a tile, fetched ahead: thread e has 8 elements of vector e % 32
    constexpr int XPT = TK * (kHeadDim / 8) >= NT ? TK * (kHeadDim / 8) / NT : 1;
    const bool stages = tid < TK * (kHeadDim / 8);     // with 1024 threads only half of them
    Raw8<XT> xr[XPT];
    const XT* xhead_base = static_cast<const XT*>(a.x) + xhead * a.x_head_stride + a.x_row0 * kHeadDim;
    auto fetch_x = [&](int64_t tile) {
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int e = tid + i * NT, k8 = e / TK;
            const int64_t row = row_of(min(tile * TK + e % TK, n_items() - 1));   // rows past the end: a stand-in, never stored
            if (stages) load_raw(xhead_base + row * kHeadDim + k8 * 8, xr[i]);
        }
    };
    bool more = true;
    while (more) {
    fetch_x(tile0);
    for (int64_t tile = tile0; tile < tile1; ++tile) {
        const int64_t r0 = tile * TK;
        const int rows = static_cast<int>(min(static_cast<int64_t>(TK), n_items() - r0));
        __syncthreads();   // the previous tile is done with LDS
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int e = tid + i * NT;
            if (stages) XTile<XT>::put(xs, e / TK, e % TK, xr[i]);
        }
        __syncthreads();
        if (tile + 1 < tile1) fetch_x(tile + 1);   // in flight during this tile

        // ---- layer 1: hidden activations
        sumsq = 0.0f;
        if constexpr (NUB > 0) {
#pragma unroll
            for (int i = 0; i < NUB; ++i) {
                ublk[i].stay_packed();
                if (wave + NW * i < nub) layer1(wave + NW * i, ublk[i]);
            }
        } else if constexpr (NUB < 0) {
            for (int ub = wave; ub < nub; ub += NW) {
                load_block(ub, ublk[0]);
                layer1(ub, ublk[0]);
            }
        }
        if constexpr (NUB != 0) __syncthreads();

        uint32_t* cbase = a.codes + xhead * a.code_head_stride + (a.code_row0 + r0) * a.W;
        if constexpr (!CERT) {
            // ---- layer 2, exact: one code word after another
            auto act = [&](int s) { return NUB == 0 ? XTile<XT>::step(xs, s, lane) : hs[s * 64 + lane]; };
            for (int word = wave; word < a.W; word += NW) {
                const WT* row = w2 + static_cast<int64_t>((31 - c) * a.W + word) * K2 + 4 * half;
                f32x16_t y;
#pragma unroll
                for (int v = 0; v < 16; ++v) y[v] = 0.0f;
                constexpr int PF = 8;   // groups of 8 weights on their way
                Raw4<WT> nx[PF];
                const int n8 = K2 / 8;
#pragma unroll
                for (int p = 0; p < PF; ++p) load_raw(row + 8 * min(p, n8 - 1), nx[p]);
                for (int g0 = 0; g0 < n8; g0 += PF) {
#pragma unroll
                    for (int p = 0; p < PF; ++p) {
                        if (g0 + p < n8) {
                            float w[4];
                            expand(nx[p], w);
                            load_raw(row + 8 * min(g0 + p + PF, n8 - 1), nx[p]);
                            to_steps(w);
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                y = __builtin_amdgcn_mfma_f32_32x32x2f32(act(4 * (g0 + p) + e), w[e], y, 0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int t = (v / 4) * 8 + half * 4 + (v % 4);
                    const unsigned long long pos = __ballot(y[v] > 0.0f);
                    if (c == 0 && t < rows) cbase[static_cast<int64_t>(t) * a.W + word] = half ? static_cast<uint32_t>(pos >> 32) : static_cast<uint32_t>(pos);
                }
            }
        } else {
            // ---- norms of the activation rows; the x tile's LDS becomes scratch
            sumsq += __shfl_xor(sumsq, 32);
            if (__ballot(sumsq == 0.0f)) {   // zeros, or did their squares underflow?  (This lane's own activations, read back.)
                uint32_t bits = 0;
                for (int ub = wave; ub < nub; ub += NW)
                    for (int v = 0; v < 16; ++v) bits |= __float_as_uint(hs[(ub * 32 + 4 * half + 8 * (v / 4) + v % 4) * TK + c]) << 1;
                bits |= __shfl_xor(bits, 32);
                sumsq = square_of(sumsq, bits);
            }
            if (half == 0) m.part[wave][c] = sumsq;
            if (tid == 0) m.count = 0;
            __syncthreads();
            if (tid < TK) {
                float s = 0.0f;
#pragma unroll
                for (int p = 0; p < NW; ++p) s += m.part[p][tid];
                m.hn[tid] = norm_of(s);
            }

            // ---- layer 2, certified: wave w owns code words w, w + NW, ...
            f32x16_t acc[NBW];
            const WT* brow[NBW];
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[nb][v] = 0.0f;
                const int word = wave + NW * nb;
                const int j = word < a.W ? (31 - c) * a.W + word : 0;
                brow[nb] = w2 + static_cast<int64_t>(j) * K2 + 8 * half;
            }
            const int n_ks = K2 / 16;
            union BFrag { bf16x8_t v; uint4 u; };
            BFrag bnext[NBW];
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) bnext[nb].u = *reinterpret_cast<const uint4*>(brow[nb]);
            for (int ks = 0; ks < n_ks; ++ks) {
                BFrag b[NBW];
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) b[nb] = bnext[nb];
                if (ks + 1 < n_ks) {   // the next step's weights are requested before this step's arithmetic
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb) bnext[nb].u = *reinterpret_cast<const uint4*>(brow[nb] + (ks + 1) * 16);
                }
                float h8[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) h8[e] = hs[(ks * 16 + 8 * half + e) * TK + c];
                bf16x8_t ahi, alo;
                split8(h8, ahi, alo);
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) {
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi, b[nb].v, acc[nb], 0, 0, 0);
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo, b[nb].v, acc[nb], 0, 0, 0);
                }
            }
            __syncthreads();   // hn is there

            const float* wn = a.wnorm + static_cast<int64_t>(whead) * a.L;   // ||W2[j]|| of this head
            const int n8 = K2 / 8;
            if constexpr (AUDIT) {
                // the chain for each of this lane's outputs: its 16 vectors share the weight row
#pragma unroll 1
                for (int nb = 0; nb < NBW; ++nb) {
                    const int word = wave + NW * nb;
                    if (word >= a.W) continue;
                    const int j = (31 - c) * a.W + word;
                    const WT* row = w2 + static_cast<int64_t>(j) * K2;
                    float yc[16];
#pragma unroll
                    for (int v = 0; v < 16; ++v) yc[v] = 0.0f;
                    for (int g = 0; g < n8; ++g) {
                        float wv[8];
                        load8(row + g * 8, wv);
#pragma unroll
                        for (int q = 0; q < 8; ++q)
#pragma unroll
                            for (int v = 0; v < 16; ++v)
                                yc[v] = __builtin_fmaf(wv[q], hs[(g * 8 + q) * TK + (v / 4) * 8 + half * 4 + (v % 4)], yc[v]);
                    }
                    const float tcol = eps * wn[j];
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int t = (v / 4) * 8 + half * 4 + (v % 4);
                        if (t >= rows) continue;
                        const float y = acc[nb][v];
                        const bool sure = settled(y, tcol, m.hn[t]);
                        const float den = wn[j] * m.hn[t];
                        const float diff = __builtin_fabsf(y - yc[v]);
                        // a NaN or an infinity on either side is never settled and is not a distance
                        const float ratio = (diff == 0.0f || !(diff < INFINITY)) ? 0.0f : (den > 0.0f ? diff / den : INFINITY);   // an infinite scale: 0
                        au_ratio = fmaxf(au_ratio, ratio);
                        au_outputs += 1;
                        au_listed += sure ? 0 : 1;
                        au_wrong += (sure && ((y > 0.0f) != (yc[v] > 0.0f))) ? 1 : 0;
                    }
                }
            }

            // ---- signs, ballot-pack, and the list of outputs too close to zero to trust
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb) {
                const int word = wave + NW * nb;
                if (word >= a.W) continue;   // uniform over the wavefront
                const float tcol = eps * wn[(31 - c) * a.W + word];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int t = (v / 4) * 8 + half * 4 + (v % 4);
                    const float y = acc[nb][v];
                    const bool sure = settled(y, tcol, m.hn[t]);
                    const unsigned long long pos = __ballot(y > 0.0f);
                    if (c == 0) m.codes[t][word] = half ? static_cast<uint32_t>(pos >> 32) : static_cast<uint32_t>(pos);
                    if (!sure && t < rows) {
                        const uint32_t at = atomicAdd(&m.count, 1u);
                        if (at < static_cast<uint32_t>(kListCap))
                            m.list[at] = static_cast<uint16_t>(t | (word << 5) | (c << 9));
                    }
                }
            }
            __syncthreads();

            // ---- recomputation with the chain of the listed outputs (of every output if the list
            // overflowed); a handful of threads with a long chain each, so the weights are fetched 32 at a time
            auto chain = [&](int j, int t) {
                constexpr int PF = 4;
                const WT* row = w2 + static_cast<int64_t>(j) * K2;
                float y = 0.0f;
                for (int g0 = 0; g0 < n8; g0 += PF) {
                    Raw8<WT> raw[PF];
#pragma unroll
                    for (int p = 0; p < PF; ++p) load_raw(row + 8 * min(g0 + p, n8 - 1), raw[p]);
#pragma unroll
                    for (int p = 0; p < PF; ++p) {
                        if (g0 + p < n8) {
                            float wv[8], hv[8];
                            expand(raw[p], wv);
#pragma unroll
                            for (int q = 0; q < 8; ++q) hv[q] = hs[((g0 + p) * 8 + q) * TK + t];
                            if constexpr (OPEN) __builtin_amdgcn_sched_barrier(0);   // all on their way before the first is waited for
#pragma unroll
                            for (int q = 0; q < 8; ++q) y = __builtin_fmaf(wv[q], hv[q], y);
                        }
                    }
                }
                return y;
            };
            auto settle = [&](int t, int word, int col) {
                const uint32_t bit = 1u << col;
                if (((m.codes[t][word] & bit) != 0) != (chain((31 - col) * a.W + word, t) > 0.0f)) atomicXor(&m.codes[t][word], bit);
            };
            const uint32_t listed = m.count;
            if (listed <= static_cast<uint32_t>(kListCap)) {
                for (uint32_t e = tid; e < listed; e += NT) settle(m.list[e] & 31, (m.list[e] >> 5) & 15, m.list[e] >> 9);
            } else {
                for (int item = tid; item < TK * a.L; item += NT) settle(item % TK, (item / TK) % a.W, 31 - (item / TK) / a.W);
            }
            __syncthreads();

            // ---- the tile's codes: rows * W consecutive words
            if constexpr (OPEN) {
                uint32_t* chead = a.codes + xhead * a.code_head_stride + a.code_row0 * a.W;
                for (int e = tid; e < rows * a.W; e += NT) chead[row_of(r0 + e / a.W) * a.W + e % a.W] = m.codes[e / a.W][e % a.W];
            } else {
                for (int e = tid; e < rows * a.W; e += NT) {
                    if constexpr (AUDIT) au_wrong += settled_wrong(a, xhead, r0 + e / a.W, cbase[e], m.codes[e / a.W][e % a.W]);
                    cbase[e] = m.codes[e / a.W][e % a.W];
                }
            }
        }
    }
    more = OPEN && walk.advance(wave, lane);
    tile1 = OPEN ? walk.tiles : tile1;
    }
    if constexpr (AUDIT) {
        const uint32_t outputs = wave_sum(au_outputs), listed = wave_sum(au_listed), wrong = wave_sum(au_wrong);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) au_ratio = fmaxf(au_ratio, __shfl_xor(au_ratio, off));
        if (lane == 0) {
            atomicAdd(&a.audit->outputs, static_cast<unsigned long long>(outputs));
            if (listed) atomicAdd(&a.audit->listed, static_cast<unsigned long long>(listed));
            if (wrong) atomicAdd(&a.audit->wrong, static_cast<unsigned long long>(wrong));
            atomicMax(&a.audit->max_ratio_bits, __float_as_uint(au_ratio));   // non-negative floats order like their bits
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The certified kernel for hidden widths up to 256 and codes up to 128 bits: everything the second layer
// needs is laid out once per tile, and a wavefront finishes its own code word alone.
//
// Hidden unit and operand row are matched so that a lane's eight accumulators of layer 1 are eight
// consecutive units.  The activations go to LDS three ways: binary32 by vector (for the recomputation),
// and hi and lo exactly as the bfloat16 instruction reads them, so that the wavefronts share one split
// instead of each splitting all activations for its own word.  Wavefront w owns code word w: it
// contracts it, takes the signs and recomputes what the bound does not settle itself, with the weights
// it holds, so a tile costs two barriers.  Two workgroups per compute unit (LDS and registers).
// Measured in one pass, 32 heads x 131072 vectors, 128 -> 256 -> 128: 4.28 ms (128 TFLOP/s), against 6.25 ms with
// layer 1 on the vector ALU (bfloat16 calls of that size take two passes now, hash_screen.h).  A tile took 19.8 K cycles
// of a SIMD (counters, before the bound became four times smaller): 8.2 K of binary32 and 1.0 K of bfloat16 matrix instructions
// and 8.1 K of vector instructions (by count SiLU 4.0 K, recomputation 1.9 K, unpacking 1.0 K), of which only the bfloat16
// ones overlap with others.  Tried and slower: a list of open outputs shared by the workgroup, one
// wavefront taking all of it (4.55 ms: fewer instructions, but everybody waits for its chain); the
// kernel below with three or four wavefronts per SIMD (4.6 and 5.0 ms); the contraction split over the
// hidden units with sums through LDS float atomics (14.7 ms: those take about 4 cycles a lane).
// hidden unit of operand row r of a block: bits 2 and 3 exchanged
__device__ __forceinline__ int unit_of_row(int r) { return (r & 19) | ((r & 4) << 1) | ((r & 8) >> 1); }

template <int NW> struct CertScratch {
    float part[NW][kTile];            // sums of squares of the wavefronts' activations
    float hn[NW][kTile];              // ||h_t||, a copy for each wavefront
    uint32_t codes[NW][kTile];
};

constexpr int hs_stride(int hidden) { return hidden_padded(hidden) + 4; }   // words per vector: b128 accesses of 8 lanes miss each other

// Operands of a step of 16 units kept in LDS: hi and lo, or with the x tile in binary32 and up to 256 units
// lo alone, so that two workgroups fit into a compute unit; hi is then taken from the activations again
// (four conversions a step).  128 -> 256 -> 128 with both kept and with lo: 512 heads x 18 binary32 vectors
// 46.8 and 31.9 us, 256 x 70 70 and 49.7 us, 8 x 30000 361 and 306 us.
template <typename XT, int NUB> constexpr int kept_operands() { return sizeof(XT) == 4 && NUB > 1 ? 1 : 2; }

// NUB: blocks of 32 hidden units a wavefront owns; WREG: steps of 16 units of layer 2.
template <typename XT, int NW, int NUB, int WREG, bool AUDIT, bool OPEN = false>
__global__ __launch_bounds__(NW * 64, 2) void hash_cert_kernel(HashArgs a, float eps, int run, int extra)
{
    using WT = bf16_raw;
    constexpr int TK = kTile, NT = NW * 64;
    extern __shared__ __align__(16) float lds[];
    float* xs = lds;                                                        // the x tile
    const int stride = hs_stride(a.hidden), nub = hidden_padded(a.hidden) / 32;
    float* hs = xs + XTile<XT>::kFloats;                                    // [TK][stride]
    constexpr int KEPT = kept_operands<XT, NUB>();
    uint4* hilo = reinterpret_cast<uint4*>(hs + TK * stride);               // [2 nub steps of 16 units][hi, lo or lo][64]
    float* bias = reinterpret_cast<float*>(hilo + nub * 2 * KEPT * 64);     // [hidden, padded to 32]
    CertScratch<NW>& m = *reinterpret_cast<CertScratch<NW>*>(bias + nub * 32);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, half = lane >> 5;
    Share share{static_cast<int>(blockIdx.y), static_cast<int64_t>(blockIdx.x) * run, run};
    if (!OPEN && extra != 0) share = share_of(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x, gridDim.y, run, extra);
    OpenJob job{};   // OPEN: in place of the share; its list is `extra` bytes into LDS
    if constexpr (OPEN) {
        job = open_job(*reinterpret_cast<OpenRows*>(reinterpret_cast<char*>(lds) + extra), a, run, wave, lane);
        if (job.parts == 0) return;
    }
    const int xhead = OPEN ? job.xhead : share.head;
    const int whead = whead_of(a, xhead);
    const WT* w1 = static_cast<const WT*>(a.w1) + static_cast<int64_t>(whead) * a.hidden * kHeadDim;
    const WT* b1 = static_cast<const WT*>(a.b1) + static_cast<int64_t>(whead) * a.hidden;
    const WT* w2 = static_cast<const WT*>(a.w2) + static_cast<int64_t>(whead) * a.L * a.hidden;
    const int n_mine = max(0, min(NUB, nub - wave * NUB));           // blocks of this wavefront
    const int n_ks = a.hidden / 16;                                  // hidden is a multiple of 16

    const int64_t n_tiles = (a.n_rows + TK - 1) / TK;
    const int64_t first = OPEN ? job.first : share.tile;
    int64_t tile0 = first, tile1 = min(n_tiles, first + (OPEN ? kOpenSegment / TK : share.tiles));
    OpenWalk walk{*reinterpret_cast<OpenRows*>(reinterpret_cast<char*>(lds) + (OPEN ? extra : 0)), OPEN ? a.open + xhead * a.open_stride + first : nullptr,
                  static_cast<int>(min(a.n_rows - first * TK, static_cast<int64_t>(kOpenSegment))), 0, 0, 0, 0, 0};
    if constexpr (OPEN) {
        if (!walk.begin(job.part, job.parts, tid, NT) || !walk.advance(wave, lane)) return;
        tile0 = 0;
        tile1 = walk.tiles;
    }
    auto n_items = [&]() { return OPEN ? static_cast<int64_t>(walk.count) : a.n_rows; };
    auto row_of = [&](int64_t item) { return OPEN ? first * TK + walk.list.row[item] : item; };

    // ---- the weights of both layers, into registers by way of LDS: read by the wavefronts as they
    // need them, a row per lane, every load touches 32 cache lines and the lines leave the cache
    // before their other parts are asked for (a workgroup with a single tile took 43 us, most of it this).
    // Rows are a multiple of 16 bytes, one chunk apart in LDS so that the rows of a wavefront miss each other.
    auto stage = [&](const WT* src, int n_rows, int chunks) {
        const uint4* from = reinterpret_cast<const uint4*>(src);
        uint4* to = reinterpret_cast<uint4*>(lds);
        constexpr int PF = 8;
        const int n = n_rows * chunks;
        for (int e0 = tid; e0 < n; e0 += NT * PF) {
            uint4 v[PF];
#pragma unroll
            for (int p = 0; p < PF; ++p) v[p] = from[min(e0 + p * NT, n - 1)];
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                const int e = e0 + p * NT;
                if (e < n) to[e / chunks * (chunks + 1) + e % chunks] = v[p];
            }
        }
    };
    const uint4* staged = reinterpret_cast<const uint4*>(lds);
    stage(w1, a.hidden, kHeadDim / 8);
    __syncthreads();
    UnitBlock<WT> ublk[NUB];   // layer 1: a row of W1 per lane, turned into the operands of the 64 steps
#pragma unroll
    for (int i = 0; i < NUB; ++i) {
        if (i >= n_mine) continue;
        const int unit = (wave * NUB + i) * 32 + unit_of_row(c);
        const uint4* row = staged + min(unit, a.hidden - 1) * (kHeadDim / 8 + 1) + half;
#pragma unroll
        for (int g = 0; g < 8; ++g) {   // k = 16 g .. + 7 in the lower half, 16 g + 8 .. + 15 in the upper
            const uint4 w = unit < a.hidden ? row[2 * g] : make_uint4(0u, 0u, 0u, 0u);
            const uint32_t d[4] = {w.x, w.y, w.z, w.w};
            float s0[4], s1[4];         // steps 8 g .. + 3 and 8 g + 4 .. + 7
#pragma unroll
            for (int p = 0; p < 4; ++p) {   // exchanges the upper half of the even k with the lower half of the odd k
                const auto r = __builtin_amdgcn_permlane32_swap(d[p] << 16, d[p] & 0xffff0000u, false, false);
                s0[p] = __uint_as_float(r[0]);
                s1[p] = __uint_as_float(r[1]);
            }
            ublk[i].put(2 * g, s0);
            ublk[i].put(2 * g + 1, s1);
        }
    }
    __syncthreads();
    stage(w2, a.L, a.hidden / 8);
    __syncthreads();
    uint4 wreg[WREG];          // layer 2: the wavefront's code word, 16 units a step, 8 of them per lane
#pragma unroll
    for (int ks = 0; ks < WREG; ++ks)
        wreg[ks] = staged[((31 - c) * a.W + min(wave, a.W - 1)) * (a.hidden / 8 + 1) + min(ks, n_ks - 1) * 2 + half];
    __syncthreads();
    for (int i = tid; i < nub * 32; i += NT) bias[i] = i < a.hidden ? load1(b1 + i) : 0.0f;

    uint32_t au_outputs = 0, au_listed = 0, au_wrong = 0;   // this lane's audit totals
    float au_ratio = 0.0f;

    // the x tile of a tile, fetched ahead: thread e has 8 elements of vector e % 32
    constexpr int XPT = TK * (kHeadDim / 8) / NT;
    Raw8<XT> xr[XPT];
    const XT* xhead_base = static_cast<const XT*>(a.x) + xhead * a.x_head_stride + a.x_row0 * kHeadDim;
    auto fetch_x = [&](int64_t tile) {
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int e = tid + i * NT;
            const int64_t row = row_of(min(tile * TK + e % TK, n_items() - 1));   // rows past the end: a stand-in, never stored
            load_raw(xhead_base + row * kHeadDim + (e / TK) * 8, xr[i]);
        }
    };
    auto put_x = [&]() {
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int e = tid + i * NT;
            XTile<XT>::put(xs, e / TK, e % TK, xr[i]);
        }
    };
    fetch_x(tile0);
    float norm = 0.0f;         // ||W2[j]|| of this lane's output
#pragma unroll
    for (int ks = 0; ks < WREG; ++ks) {
        if (ks >= n_ks) continue;
        const uint32_t d[4] = {wreg[ks].x, wreg[ks].y, wreg[ks].z, wreg[ks].w};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const float lo = __uint_as_float(d[p] << 16), hi = __uint_as_float(d[p] & 0xffff0000u);
            norm = __builtin_fmaf(hi, hi, __builtin_fmaf(lo, lo, norm));
        }
    }
    norm += __shfl_xor(norm, 32);
    if (rare(norm == 0.0f))   // a row of zeros, or did its squares underflow?
        norm = square_of(norm, magnitude_bits(w2 + static_cast<int64_t>((31 - c) * a.W + min(wave, a.W - 1)) * a.hidden, a.hidden));
    norm = norm_of(norm);
    bool more = true;
    while (more) {
    put_x();
    __syncthreads();
    for (int64_t tile = tile0; tile < tile1; ++tile) {
        const int64_t r0 = tile * TK;
        const int rows = static_cast<int>(min(static_cast<int64_t>(TK), n_items() - r0));
        if (tile + 1 < tile1) fetch_x(tile + 1);   // in flight during layer 1

        // ---- layer 1.  The SiLU of a block runs in the shadow of the next block's matrix instructions.
        f32x16_t h[NUB];
        float sumsq = 0.0f;
        auto activate = [&](int i, int v) {
            h[i][v] = silu(h[i][v]);
            sumsq = __builtin_fmaf(h[i][v], h[i][v], sumsq);
        };
        auto keep = [&](int i, int j) {   // accumulators 8 j .. 8 j + 7: units 16 j + 8 half .. + 7 of the block
            float h8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) h8[e] = h[i][8 * j + e];
            const int ub = wave * NUB + i;
            float4* f = reinterpret_cast<float4*>(hs + c * stride + ub * 32 + 16 * j + 8 * half);
            f[0] = make_float4(h8[0], h8[1], h8[2], h8[3]);
            f[1] = make_float4(h8[4], h8[5], h8[6], h8[7]);
            bf16x8_t hi, lo;
            split8(h8, hi, lo);
            if constexpr (KEPT == 2) hilo[((ub * 2 + j) * 2 + 0) * 64 + lane] = __builtin_bit_cast(uint4, hi);
            hilo[((ub * 2 + j) * KEPT + KEPT - 1) * 64 + lane] = __builtin_bit_cast(uint4, lo);
        };
#pragma unroll
        for (int i = 0; i < NUB; ++i) {
            ublk[i].stay_packed();
            if (i >= n_mine) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {   // accumulators 4 q .. 4 q + 3
                const float4 f = *reinterpret_cast<const float4*>(bias + (wave * NUB + i) * 32 + 16 * (q / 2) + 8 * half + 4 * (q % 2));
                h[i][4 * q] = f.x; h[i][4 * q + 1] = f.y; h[i][4 * q + 2] = f.z; h[i][4 * q + 3] = f.w;
            }
#pragma unroll
            for (int s = 0; s < kHeadDim / 2; ++s) {
                h[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(ublk[i].step(s), XTile<XT>::step(xs, s, lane), h[i], 0, 0, 0);
                if (i > 0 && s % 4 == 3) activate(i - 1, s / 4);
                if (i > 0 && s % 32 == 31) keep(i - 1, s / 32);
            }
        }
#pragma unroll
        for (int i = 0; i < NUB; ++i) {
            if (i == n_mine - 1) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    activate(i, v);
                    if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // four at a time: sixteen side by side would spill
                }
                keep(i, 0);
                keep(i, 1);
            }
        }
        sumsq += __shfl_xor(sumsq, 32);
        if (half == 0) m.part[wave][c] = sumsq;
        __syncthreads();   // activations and norms are complete; the x tile is free
        if (tile + 1 < tile1) put_x();

        // ---- layer 2 of this wavefront's word
        if (wave < a.W) {
            float s = 0.0f;
#pragma unroll
            for (int p = 0; p < NW; ++p) s += m.part[p][c];
            if (rare(s == 0.0f)) {   // zeros, or did their squares underflow?
                uint32_t bits = 0;
#pragma unroll 1
                for (int i = 4 * half; i < a.hidden; i += 8) bits |= magnitude_bits(*reinterpret_cast<const float4*>(hs + c * stride + i));
                s = square_of(s, bits | __shfl_xor(bits, 32));
            }
            if (half == 0) m.hn[wave][c] = norm_of(s);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

            f32x16_t y;
#pragma unroll
            for (int v = 0; v < 16; ++v) y[v] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < WREG; ++ks) {
                if (ks >= n_ks) continue;
                uint4 hi, lo = hilo[(ks * KEPT + KEPT - 1) * 64 + lane];
                if constexpr (KEPT == 2) {
                    hi = hilo[ks * 2 * 64 + lane];
                } else {
                    const float4* f = reinterpret_cast<const float4*>(hs + c * stride + ks * 16 + 8 * half);
                    hi = round8(f[0], f[1]);
                }
                y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, hi), __builtin_bit_cast(bf16x8_t, wreg[ks]), y, 0, 0, 0);
                y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, lo), __builtin_bit_cast(bf16x8_t, wreg[ks]), y, 0, 0, 0);
            }

            float hn[16];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 f = *reinterpret_cast<const float4*>(&m.hn[wave][8 * q + 4 * half]);
                hn[4 * q] = f.x; hn[4 * q + 1] = f.y; hn[4 * q + 2] = f.z; hn[4 * q + 3] = f.w;
            }
            {
                const int word = wave;
                const float tcol = eps * norm;

                if constexpr (AUDIT) {   // the chain for each of this lane's outputs
                    const WT* row = w2 + static_cast<int64_t>((31 - c) * a.W + word) * a.hidden;
#pragma unroll 1
                    for (int v = 0; v < 16; ++v) {
                        const int t = (v / 4) * 8 + half * 4 + (v % 4);
                        float yc = 0.0f, yv = 0.0f, hv = 0.0f;
#pragma unroll
                        for (int e = 0; e < 16; ++e) { yv = e == v ? y[e] : yv; hv = e == v ? hn[e] : hv; }
                        for (int g = 0; g < a.hidden / 8; ++g) {
                            float wv[8];
                            load8(row + g * 8, wv);
#pragma unroll
                            for (int e = 0; e < 8; ++e) yc = __builtin_fmaf(wv[e], hs[t * stride + g * 8 + e], yc);
                        }
                        if (t >= rows) continue;
                        const bool sure = settled(yv, tcol, hv);
                        const float den = norm * hv, diff = __builtin_fabsf(yv - yc);
                        // a NaN or an infinity on either side is never settled and is not a distance
                        const float ratio = (diff == 0.0f || !(diff < INFINITY)) ? 0.0f : (den > 0.0f ? diff / den : INFINITY);   // an infinite scale: 0
                        au_ratio = fmaxf(au_ratio, ratio);
                        au_outputs += 1;
                        au_listed += sure ? 0 : 1;
                        au_wrong += (sure && ((yv > 0.0f) != (yc > 0.0f))) ? 1 : 0;
                    }
                }

                // ---- signs, packed by ballots; a lane notes which of its 16 outputs are too close to zero to trust
                uint32_t open = 0;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int t = (v / 4) * 8 + half * 4 + (v % 4);
                    const bool sure = settled(y[v], tcol, hn[v]);
                    const unsigned long long pos = __ballot(y[v] > 0.0f);
                    if (c == 0) m.codes[wave][t] = half ? static_cast<uint32_t>(pos >> 32) : static_cast<uint32_t>(pos);
                    open |= sure ? 0u : 1u << v;
                }
                if (rows < TK) {   // rows past the end are copies of the last one: not to be recomputed over and over
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if ((v / 4) * 8 + half * 4 + (v % 4) >= rows) open &= ~(1u << v);
                }
                // ---- recomputation with the chain, a round for every lane's next open output (nearly always
                // one round).  A lane's output row is the one it has the weights of: its own 8 of 16 units
                // are here, the other 8 are in the other half.
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                while (__ballot(open != 0)) {
                    const int v = open ? __builtin_ctz(open) : 0;
                    const int t = (v / 4) * 8 + half * 4 + (v % 4);
                    const float* hr = hs + t * stride;
                    float yc = 0.0f;
#pragma unroll
                    for (int ks = 0; ks < WREG; ++ks) {
                        if (ks >= n_ks) continue;
                        const uint32_t own[4] = {wreg[ks].x, wreg[ks].y, wreg[ks].z, wreg[ks].w};
                        uint32_t first[4], second[4];   // units 16 ks .. + 7 and 16 ks + 8 .. + 15, in both halves
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const auto r = __builtin_amdgcn_permlane32_swap(own[e], own[e], false, false);
                            first[e] = r[0];
                            second[e] = r[1];
                        }
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            const float4 f = *reinterpret_cast<const float4*>(hr + ks * 16 + 4 * p);
                            const uint32_t wa = p < 2 ? first[2 * p] : second[2 * p - 4], wb = p < 2 ? first[2 * p + 1] : second[2 * p - 3];
                            yc = __builtin_fmaf(__uint_as_float(wa << 16), f.x, yc);
                            yc = __builtin_fmaf(__uint_as_float(wa & 0xffff0000u), f.y, yc);
                            yc = __builtin_fmaf(__uint_as_float(wb << 16), f.z, yc);
                            yc = __builtin_fmaf(__uint_as_float(wb & 0xffff0000u), f.w, yc);
                        }
                    }
                    if (open) {
                        const uint32_t bit = 1u << c;
                        if (((m.codes[wave][t] & bit) != 0) != (yc > 0.0f)) atomicXor(&m.codes[wave][t], bit);
                        open &= open - 1;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (lane < rows) {
                    uint32_t* to = a.codes + xhead * a.code_head_stride + (a.code_row0 + row_of(r0 + lane)) * a.W + word;
                    if constexpr (AUDIT) au_wrong += settled_wrong(a, xhead, r0 + lane, *to, m.codes[wave][lane]);
                    *to = m.codes[wave][lane];
                }
            }
        }
        __syncthreads();   // LDS may be written again
    }
    more = OPEN && walk.advance(wave, lane);
    if (more) {
        tile1 = walk.tiles;
        fetch_x(0);
    }
    }
    if constexpr (AUDIT) {
        const uint32_t outputs = wave_sum(au_outputs), listed = wave_sum(au_listed), wrong = wave_sum(au_wrong);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) au_ratio = fmaxf(au_ratio, __shfl_xor(au_ratio, off));
        if (lane == 0) {
            atomicAdd(&a.audit->outputs, static_cast<unsigned long long>(outputs));
            if (listed) atomicAdd(&a.audit->listed, static_cast<unsigned long long>(listed));
            if (wrong) atomicAdd(&a.audit->wrong, static_cast<unsigned long long>(wrong));
            atomicMax(&a.audit->max_ratio_bits, __float_as_uint(au_ratio));   // non-negative floats order like their bits
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The linear hash sign(xR) with bfloat16 weights, certified as above (eps with 128 in place of hidden).
//
// With nothing in front of it the contraction needs no binary32 matrix instruction at all: bfloat16
// vectors enter the matrix cores as they are, binary32 ones as hi + lo.  A wavefront keeps the weights
// of up to four code words in registers and streams tiles of 32 vectors from LDS, already in operand
// order, double-buffered with one barrier a tile.  What is left is the vector work of the signs (about
// six instructions for 64 outputs) and waits: 65536 x 8 vectors of 512 bits went from 983 us on the vector ALU
// (728 us on the binary32 matrix instruction) to 270 us; 39 % of the cycles issue vector instructions, 10 %
// are matrix instructions (221 us with the smaller bound; calls of that size go to the next kernel now).  With four words a wavefront 50 registers are spilled (66 with binary32 vectors); a
// recomputation that holds half as many operands spills 48 and is slower (284 us).
constexpr int kLinearWords = 16;      // code words of a workgroup, four a wavefront here (longer codes have the next kernel)
constexpr int kLinearList = 256;      // open outputs of a wavefront and tile (of 32 x 128)
constexpr int kLinearStage = 256;     // rows of R on their way into registers at a time

template <typename XT> struct LinearLds {
    static constexpr int kPasses = sizeof(XT) == 2 ? 1 : 2;     // hi, or hi and lo
    uint4 x[2][kPasses][16 * kTile];                            // [chunk of 8 k][vector, exclusive-or with the chunk]
    float hn[2][kTile];                                         // ||x_t||
    uint32_t codes[2][kTile][kLinearWords];
    uint16_t list[4][kLinearList];
    uint4 pad;                                                  // the staging of R may run over the end of the rest
};

// NB: code words of a wavefront
template <typename XT, int NB, bool AUDIT>
__global__ __launch_bounds__(kThreads, 2) void hash_linear_kernel(HashArgs a, float eps, int tiles_per_group)
{
    using WT = bf16_raw;
    constexpr int TK = kTile, NT = kThreads, CH = kHeadDim / 8;
    constexpr int PASSES = LinearLds<XT>::kPasses;
    extern __shared__ __align__(16) float lds[];
    LinearLds<XT>& m = *reinterpret_cast<LinearLds<XT>*>(lds);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, half = lane >> 5;
    const int xhead = blockIdx.y;
    const int whead = whead_of(a, xhead);
    const int n_words = a.W;
    const WT* r = static_cast<const WT*>(a.w1) + static_cast<int64_t>(whead) * a.L * kHeadDim;
    const XT* xbase = static_cast<const XT*>(a.x) + xhead * a.x_head_stride + a.x_row0 * kHeadDim;

    // ---- R into registers by way of LDS (whole cache lines), kLinearStage rows at a time: word
    // wave + 4 nb, the lane's output, 16 k a step and 8 of them per lane
    uint4 wreg[NB][8];
    for (int j0 = 0; j0 < a.L; j0 += kLinearStage) {
        const uint4* from = reinterpret_cast<const uint4*>(r + static_cast<int64_t>(j0) * kHeadDim);
        uint4* to = reinterpret_cast<uint4*>(lds);
        const int rows = min(kLinearStage, a.L - j0), n = rows * CH;
        for (int e0 = tid; e0 < n; e0 += NT * 8) {
            uint4 v[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) v[p] = from[min(e0 + p * NT, n - 1)];
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int e = e0 + p * NT;
                if (e < n) to[e / CH * (CH + 1) + e % CH] = v[p];
            }
        }
        __syncthreads();
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int j = (31 - c) * a.W + min(wave + 4 * nb, n_words - 1) - j0;
            if (j >= 0 && j < rows) {
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) wreg[nb][ks] = reinterpret_cast<const uint4*>(lds)[j * (CH + 1) + 2 * ks + half];
            }
        }
        __syncthreads();
    }
    uint32_t au_outputs = 0, au_listed = 0, au_wrong = 0;   // this lane's audit totals
    float au_ratio = 0.0f;

    const int64_t n_tiles = (a.n_rows + TK - 1) / TK;
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * tiles_per_group;
    const int64_t tile1 = min(n_tiles, tile0 + tiles_per_group);

    // 16 neighbouring threads have one vector, 8 elements each
    constexpr int XPT = TK * CH / NT;
    Raw8<XT> xr[XPT];
    auto fetch_x = [&](int64_t tile) {
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int e = tid + i * NT;
            const int64_t row = min(tile * TK + e / CH, a.n_rows - 1);   // rows past the end: a stand-in, never stored
            load_raw(xbase + row * kHeadDim + (e % CH) * 8, xr[i]);
        }
    };
    auto put_x = [&](int buf) {
        float s[XPT];
        bool none = false;
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int e = tid + i * NT, t = e / CH, k8 = e % CH, at = k8 * TK + (t ^ k8);
            float v[8];
            expand(xr[i], v);
            if constexpr (PASSES == 1) {
                m.x[buf][0][at] = xr[i].u;
            } else {
                bf16x8_t hi, lo;
                split8(v, hi, lo);
                m.x[buf][0][at] = __builtin_bit_cast(uint4, hi);
                m.x[buf][PASSES - 1][at] = __builtin_bit_cast(uint4, lo);
            }
            s[i] = 0.0f;
#pragma unroll
            for (int q = 0; q < 8; ++q) s[i] = __builtin_fmaf(v[q], v[q], s[i]);
            s[i] = add_across_16(s[i]);
            none = none || s[i] == 0.0f;
        }
        // zeros, or did their squares underflow?  (Both sums first: a branch behind each costs a launch of single tiles
        // 1 us.  Looked at only where outputs turn out to be open, which is in nearly every tile: 263 -> 301 us for
        // 8 x 65536 vectors of 512 bits, this way 267.)
        if (rare(none)) {
#pragma unroll
            for (int i = 0; i < XPT; ++i)
                s[i] = square_of(s[i], static_cast<uint32_t>(__ballot(magnitude_bits(xr[i]) != 0) >> (lane & 48)) & 0xffffu);
        }
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int e = tid + i * NT;
            if (e % CH == 0) m.hn[buf][e / CH] = norm_of(s[i]);
        }
    };
    // the chain of output row j for vector `row`, from the arrays as stored
    auto chain = [&](int64_t row, int j) {
        const XT* xp = xbase + row * kHeadDim;
        const WT* rp = r + static_cast<int64_t>(j) * kHeadDim;
        float y = 0.0f;
#pragma unroll 1
        for (int g0 = 0; g0 < CH; g0 += 4) {
            Raw8<XT> xv[4];
            Raw8<WT> wv[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) { load_raw(xp + (g0 + p) * 8, xv[p]); load_raw(rp + (g0 + p) * 8, wv[p]); }
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                float xf[8], wf[8];
                expand(xv[p], xf);
                expand(wv[p], wf);
#pragma unroll
                for (int q = 0; q < 8; ++q) y = __builtin_fmaf(wf[q], xf[q], y);
            }
        }
        return y;
    };

    fetch_x(tile0);
    float tcol[NB];   // eps ||R_j||
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float s = 0.0f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const uint32_t d[4] = {wreg[nb][ks].x, wreg[nb][ks].y, wreg[nb][ks].z, wreg[nb][ks].w};
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const float lo = __uint_as_float(d[p] << 16), hi = __uint_as_float(d[p] & 0xffff0000u);
                s = __builtin_fmaf(hi, hi, __builtin_fmaf(lo, lo, s));
            }
        }
        s += __shfl_xor(s, 32);
        if (rare(s == 0.0f))   // a row of zeros, or did its squares underflow?
            s = square_of(s, magnitude_bits(r + static_cast<int64_t>((31 - c) * a.W + min(wave + 4 * nb, n_words - 1)) * kHeadDim, kHeadDim));
        tcol[nb] = eps * norm_of(s);
    }
    put_x(0);
    if (tile0 + 1 < tile1) fetch_x(tile0 + 1);
    __syncthreads();
    for (int64_t tile = tile0; tile < tile1; ++tile) {
        const int buf = static_cast<int>(tile - tile0) & 1;
        const int64_t r0 = tile * TK;
        const int rows = static_cast<int>(min(static_cast<int64_t>(TK), a.n_rows - r0));
        if (tile + 1 < tile1) put_x(buf ^ 1);
        if (tile + 2 < tile1) fetch_x(tile + 2);

        float hn[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 f = *reinterpret_cast<const float4*>(&m.hn[buf][8 * q + 4 * half]);
            hn[4 * q] = f.x; hn[4 * q + 1] = f.y; hn[4 * q + 2] = f.z; hn[4 * q + 3] = f.w;
        }
        // ---- signs, packed by ballots, and the wavefront's list of outputs too close to zero to trust
        uint32_t listed = 0;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int w = wave + 4 * nb;
            if (w >= n_words) continue;   // uniform over the wavefront
            f32x16_t y;                   // one word at a time: registers are short as it is, and the vector unit is what is busy
#pragma unroll
            for (int v = 0; v < 16; ++v) y[v] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
#pragma unroll
                for (int p = 0; p < PASSES; ++p) {
                    const int k8 = 2 * ks + half;
                    const uint4 x = m.x[buf][p][k8 * TK + (c ^ k8)];
                    y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, wreg[nb][ks]), y, 0, 0, 0);
                }
            if constexpr (AUDIT) {
#pragma unroll 1
                for (int v = 0; v < 16; ++v) {
                    const int t = (v / 4) * 8 + half * 4 + (v % 4);
                    if (t >= rows) continue;
                    float yv = 0.0f, hv = 0.0f;
#pragma unroll
                    for (int e = 0; e < 16; ++e) { yv = e == v ? y[e] : yv; hv = e == v ? hn[e] : hv; }
                    const float yc = chain(r0 + t, (31 - c) * a.W + w);
                    const bool sure = settled(yv, tcol[nb], hv);
                    const float den = tcol[nb] / eps * hv, diff = __builtin_fabsf(yv - yc);
                    // a NaN or an infinity on either side is never settled and is not a distance
                    const float ratio = (diff == 0.0f || !(diff < INFINITY)) ? 0.0f : (den > 0.0f ? diff / den : INFINITY);   // an infinite scale: 0
                    au_ratio = fmaxf(au_ratio, ratio);
                    au_outputs += 1;
                    au_listed += sure ? 0 : 1;
                    au_wrong += (sure && ((yv > 0.0f) != (yc > 0.0f))) ? 1 : 0;
                }
            }
            unsigned long long any = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = (v / 4) * 8 + half * 4 + (v % 4);
                const unsigned long long pos = __ballot(y[v] > 0.0f);
                any |= __ballot(!settled(y[v], tcol[nb], hn[v]));
                if (c == 0) m.codes[buf][t][w] = half ? static_cast<uint32_t>(pos >> 32) : static_cast<uint32_t>(pos);
            }
            if (any) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int t = (v / 4) * 8 + half * 4 + (v % 4);
                    const bool open = t < rows && !settled(y[v], tcol[nb], hn[v]);
                    const unsigned long long o = __ballot(open);
                    if (o) {
                        const uint32_t at = listed + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(o >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(o), 0u));
                        if (open && at < static_cast<uint32_t>(kLinearList)) m.list[wave][at] = static_cast<uint16_t>(t | (c << 5) | (nb << 10));
                        listed += static_cast<uint32_t>(__builtin_popcountll(o));
                    }
                }
            }
        }
        // ---- recomputation with the chain, a lane each (of everything the wavefront has if the list overflowed)
        if (listed) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const bool all = listed > static_cast<uint32_t>(kLinearList);
            const uint32_t n = all ? static_cast<uint32_t>(NB * TK * 32) : listed;
            for (uint32_t e = lane; e < n; e += 64) {
                const int entry = all ? static_cast<int>(e) : m.list[wave][e];
                const int t = entry & 31, col = (entry >> 5) & 31, w = wave + 4 * (entry >> 10);
                if (t >= rows || w >= n_words) continue;
                const float yc = chain(r0 + t, (31 - col) * a.W + w);
                const uint32_t bit = 1u << col;
                if (((m.codes[buf][t][w] & bit) != 0) != (yc > 0.0f)) atomicXor(&m.codes[buf][t][w], bit);
            }
        }
        __syncthreads();   // the tile's codes are final, the next tile's vectors are there
        uint32_t* cbase = a.codes + xhead * a.code_head_stride + (a.code_row0 + r0) * a.W;
        for (int e = tid; e < rows * n_words; e += NT) cbase[static_cast<int64_t>(e / n_words) * a.W + e % n_words] = m.codes[buf][e / n_words][e % n_words];
    }
    if constexpr (AUDIT) {
        const uint32_t outputs = wave_sum(au_outputs), listed = wave_sum(au_listed), wrong = wave_sum(au_wrong);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) au_ratio = fmaxf(au_ratio, __shfl_xor(au_ratio, off));
        if (lane == 0) {
            atomicAdd(&a.audit->outputs, static_cast<unsigned long long>(outputs));
            if (listed) atomicAdd(&a.audit->listed, static_cast<unsigned long long>(listed));
            if (wrong) atomicAdd(&a.audit->wrong, static_cast<unsigned long long>(wrong));
            atomicMax(&a.audit->max_ratio_bits, __float_as_uint(au_ratio));   // non-negative floats order like their bits
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The same for larger calls.  R is in LDS as the instruction reads it (128 KB for
// 512 bits), rows = the outputs of a word, columns = vectors; a wavefront takes two tiles of 32 vectors alone (one of
// binary32), straight from memory into its registers, and all words of them, so that an operand of R feeds two
// instructions and nothing waits at a barrier.  Lane c + 32 half has outputs 16 half .. 16 half + 15 of a word of vector c: the
// code is shifted together from the signs, and one comparison of the smallest of them with the word's largest bound tells
// whether the word is settled (where the rows of a word are uneven and that does not, each output is held to the bound of its own
// row: one row of 32 a hundred or a thousand times the others, 148 and 755 us without, 137 with; ten times 98 without, 111 with).  Outputs
// that are not (3 in 100000) go to a list of the wavefront, whose chains run when it is full or
// the work is done, a lane each, and correct the codes in memory.
// 8 heads x 65536 vectors of 512 bits: 221 us with the kernel above (waits for operands, barriers and chains),
// 87 us; 32 x 65536 of 128 bits 467 and 132 us; binary32 vectors of 512 bits 322 and 146 us.
constexpr int kLinearWaves = 8;       // wavefronts of a workgroup
constexpr int kTilesList = 192;       // open outputs a wavefront keeps; at most 64 come at a time
constexpr float kUneven = 32.0f;      // rows of a word are uneven where one bound for all leaves more than this many times the outputs open

// How often the product of index j counts in the bound: n / 2 sums of the chain and three times as many groups' sums as are
// added up to the nearer end, the cut products, the split (bulk_hash_eps, with each term's own share).
template <int PASSES> __device__ __forceinline__ float linear_charge(int j)
{
    const int chain = j < kHeadDim / 2 ? kHeadDim / 2 - j : j - kHeadDim / 2 + 1;
    return PASSES == 1 ? 1.375f * chain + 16.0f : 1.75f * chain + 151.0f;
}

struct LinearWord {
    float scale;                      // max_j u ||charge R_j|| over the outputs of the word
    uint32_t zeros;                   // bit c: output c * W + word has a row of zeros (y = 0, bit 0)
};
// LDS: the operands of the words in use ([8][64] of 16 bytes each), behind the operands: LinearWord[kLinearWords], each row's u ||charge R_j||
// ([kLinearWords][32] floats in the order of a word's bits) and whether they are uneven ([kLinearWords]), list[kLinearWaves][kTilesList]
inline size_t linear_lds(int words)
{
    return static_cast<size_t>(words) * 8 * 64 * sizeof(uint4) + kLinearWords * (sizeof(LinearWord) + 33 * sizeof(float)) + kLinearWaves * kTilesList * sizeof(uint32_t);
}

// the value of lane l + 32 in lane l and the other way round
__device__ __forceinline__ uint32_t other_half(uint32_t v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);   // the lower half's value in all lanes, the upper half's
    return (threadIdx.x & 32) ? r[0] : r[1];
}
__device__ __forceinline__ float add_halves(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <typename XT, bool AUDIT>
__global__ __launch_bounds__(kLinearWaves * 64, 2) void hash_linear_tiles_kernel(HashArgs a, int rounds)
{
    using WT = bf16_raw;
    constexpr int TK = kTile, CH = kHeadDim / 8;
    constexpr int PASSES = sizeof(XT) == 2 ? 1 : 2;           // hi, or hi and lo
    constexpr int KT = sizeof(XT) == 2 ? 2 : 1;               // tiles a wavefront takes together
    extern __shared__ __align__(16) float lds[];
    uint4* ops = reinterpret_cast<uint4*>(lds);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, half = lane >> 5;
    const int xhead = blockIdx.y;
    const int whead = whead_of(a, xhead);
    const int word0 = blockIdx.z * kLinearWords, n_words = min(kLinearWords, a.W - word0);
    LinearWord* lw = reinterpret_cast<LinearWord*>(ops + min(kLinearWords, a.W) * 8 * 64);
    float* row_scale = reinterpret_cast<float*>(lw + kLinearWords);
    uint32_t* uneven = reinterpret_cast<uint32_t*>(row_scale + kLinearWords * 32);
    uint32_t* list = uneven + kLinearWords + wave * kTilesList;
    const WT* r = static_cast<const WT*>(a.w1) + static_cast<int64_t>(whead) * a.L * kHeadDim;
    const XT* xbase = static_cast<const XT*>(a.x) + xhead * a.x_head_stride + a.x_row0 * kHeadDim;

    // vectors: the lane's 8 of every 16 elements of vector c of each tile
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * rounds * (kLinearWaves * KT * TK) + wave * (KT * TK);   // of this wavefront's first
    Raw8<XT> xr[KT][8];
    auto fetch_x = [&](int64_t row) {
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            const int64_t at = min(row + t * TK + c, a.n_rows - 1);   // rows past the end: a stand-in, never stored
#pragma unroll
            for (int s = 0; s < 8; ++s) load_raw(xbase + at * kHeadDim + (2 * s + half) * 8, xr[t][s]);
        }
    };
    fetch_x(row0);
    // ---- R into LDS, and its rows' norms.  Row c of an operand is the output whose bit a lane shifts in there.
    const int bit_of_row = (c >> 3) * 4 + (c & 3) + 16 * ((c >> 2) & 1);
    for (int w = wave; w < n_words; w += kLinearWaves) {
        const WT* row = r + static_cast<int64_t>(bit_of_row * a.W + word0 + w) * kHeadDim;
        uint4 v[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = *reinterpret_cast<const uint4*>(row + (2 * s + half) * 8);
        float sum = 0.0f;
        uint32_t bits = 0;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            ops[(w * 8 + s) * 64 + lane] = v[s];
            bits |= magnitude_bits(v[s]);
            const uint32_t d[4] = {v[s].x, v[s].y, v[s].z, v[s].w};
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int k = (2 * s + half) * 8 + 2 * p;
                const float lo = linear_charge<PASSES>(k) * __uint_as_float(d[p] << 16), hi = linear_charge<PASSES>(k + 1) * __uint_as_float(d[p] & 0xffff0000u);
                sum = __builtin_fmaf(hi, hi, __builtin_fmaf(lo, lo, sum));
            }
        }
        sum = add_halves(sum);
        bits |= other_half(bits);
        float norm = norm_of(square_of(sum, bits));
        const float own = norm;
        uint32_t zeros = bits == 0 ? 1u << bit_of_row : 0u;
        if (half == 0) row_scale[w * 32 + bit_of_row] = static_cast<float>(1.02 * 0x1p-24) * norm;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const float n2 = __shfl_xor(norm, off);
            norm = n2 > norm || n2 != n2 ? n2 : norm;   // a NaN stays
            zeros |= __shfl_xor(zeros, off);
        }
        float share = bits == 0 ? 0.0f : norm / own;   // how many times more outputs the largest bound leaves open than each row's own
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) share += __shfl_xor(share, off);
        if (lane == 0) { lw[w] = {static_cast<float>(1.02 * 0x1p-24) * norm, zeros}; uneven[w] = !(share <= 32.0f * kUneven); }   // also where one is no number
    }
    uint32_t au_outputs = 0, au_listed = 0, au_wrong = 0;   // this lane's audit totals
    float au_ratio = 0.0f;

    // the chain of output row j for vector `row`, from the arrays as stored; the square of the row's norm beside it
    auto chain = [&](int64_t row, int j, float& square) {
        const XT* xp = xbase + row * kHeadDim;
        const WT* rp = r + static_cast<int64_t>(j) * kHeadDim;
        float y = 0.0f;
        square = 0.0f;
#pragma unroll 1
        for (int g0 = 0; g0 < CH; g0 += 4) {
            Raw8<XT> xv[4];
            Raw8<WT> wv[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) { load_raw(xp + (g0 + p) * 8, xv[p]); load_raw(rp + (g0 + p) * 8, wv[p]); }
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                float xf[8], wf[8];
                expand(xv[p], xf);
                expand(wv[p], wf);
#pragma unroll
                for (int q = 0; q < 8; ++q) y = __builtin_fmaf(wf[q], xf[q], y);
                if constexpr (AUDIT) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) square = __builtin_fmaf(wf[q], wf[q], square);
                }
            }
        }
        return y;
    };
    // whether an output is further from zero than the bound of its own row
    auto sure_of = [&](float y, float scale, float norm) {
        const float b = scale * norm;
        return __builtin_fabsf(y) >= b && b < 1e25f;   // neither where it is no number
    };
    // ---- the list: row behind row0 << 11 | the sign as stored << 10 | word << 5 | bit
    int listed = 0;
    auto settle_list = [&]() {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // the codes are stored, the list is written
        for (int e = lane; e < listed; e += 64) {
            const uint32_t entry = list[e];
            const int64_t row = row0 + (entry >> 11);
            const int bit = entry & 31, w = (entry >> 5) & 31;
            float unused;
            const bool one = chain(row, (31 - bit) * a.W + word0 + w, unused) > 0.0f;
            // (nobody but this wavefront writes the word)
            if (one != ((entry >> 10) & 1))
                __hip_atomic_fetch_xor(a.codes + xhead * a.code_head_stride + (a.code_row0 + row) * a.W + word0 + w, 1u << bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        listed = 0;
    };
    __syncthreads();

    for (int round = 0; round < rounds; ++round) {
        const int64_t row = row0 + static_cast<int64_t>(round) * (kLinearWaves * KT * TK);
        if (row >= a.n_rows) break;
        // ---- norms, and the vectors as operands
        bf16x8_t x[KT][PASSES][8];
        float xn[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            float sum = 0.0f;
            uint32_t bits = 0;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                float v[8];
                expand(xr[t][s], v);
#pragma unroll
                for (int q = 0; q < 8; ++q) sum = __builtin_fmaf(v[q], v[q], sum);
                if constexpr (PASSES == 1) {
                    x[t][0][s] = __builtin_bit_cast(bf16x8_t, xr[t][s]);
                } else {
                    split8(v, x[t][0][s], x[t][PASSES - 1][s]);
                }
                bits |= magnitude_bits(xr[t][s]);
            }
            xn[t] = norm_of(square_of(add_halves(sum), bits | other_half(bits)));
        }
        if (round + 1 < rounds) fetch_x(row + kLinearWaves * KT * TK);   // in flight during this round
        // ---- the words, four at a time
        for (int w0 = 0; w0 < n_words; w0 += 4) {
            uint32_t code[KT][4];
#pragma unroll
            for (int wi = 0; wi < 4; ++wi) {
                const int w = min(w0 + wi, n_words - 1);
                const LinearWord word = lw[w];
                f32x16_t y[KT];
#pragma unroll
                for (int t = 0; t < KT; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) y[t][v] = 0.0f;
                if (word.zeros) {   // rows of zeros: far from zero, and negative
#pragma unroll
                    for (int t = 0; t < KT; ++t)
#pragma unroll
                        for (int v = 0; v < 16; ++v) y[t][v] = (word.zeros >> (v + 16 * half)) & 1 ? -1e30f : 0.0f;
                }
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const bf16x8_t b = __builtin_bit_cast(bf16x8_t, ops[(w * 8 + s) * 64 + lane]);
#pragma unroll
                    for (int t = 0; t < KT; ++t)
#pragma unroll
                        for (int p = 0; p < PASSES; ++p) y[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, x[t][p][s], y[t], 0, 0, 0);
                }
                float bound[KT];
                bool open = false;
#pragma unroll
                for (int t = 0; t < KT; ++t) {
                    uint32_t sign = 0;
                    float nearest = INFINITY;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        sign = __builtin_amdgcn_alignbit(sign, __float_as_uint(y[t][v]), 31);
                        nearest = fminf(nearest, __builtin_fabsf(y[t][v]));
                    }
                    bound[t] = word.scale * xn[t];
                    if (!(bound[t] < 1e25f)) bound[t] = INFINITY;                  // also where it is no number
                    open = open || (!(nearest >= bound[t]) || bound[t] == INFINITY);
                    code[t][wi] = xn[t] == 0.0f ? 0u : ~sign & 0xffffu;            // a settled output is no zero, but for a vector of zeros
                }
                if constexpr (AUDIT) {
                    if (w0 + wi < n_words) {
#pragma unroll 1
                        for (int tv = 0; tv < KT * 16; ++tv) {
                            float yv = 0.0f, xv = 0.0f;
#pragma unroll
                            for (int t = 0; t < KT; ++t)
#pragma unroll
                                for (int v = 0; v < 16; ++v) { const bool is = t * 16 + v == tv; yv = is ? y[t][v] : yv; xv = is ? xn[t] : xv; }
                            const int bit = 31 - (tv % 16 + 16 * half);
                            const int64_t at = row + tv / 16 * TK + c;
                            if (at >= a.n_rows) continue;
                            float square;
                            const float yc = chain(at, (31 - bit) * a.W + word0 + w, square);
                            const bool sure = sure_of(yv, uneven[w] ? row_scale[w * 32 + tv % 16 + 16 * half] : word.scale, xv), one = yv > 0.0f && xv != 0.0f;
                            // a NaN or an infinity on either side is never settled and is not a distance; nor is a row of zeros
                            const float den = __builtin_sqrtf(square) * xv, diff = __builtin_fabsf(yv - yc);
                            const float ratio = (diff == 0.0f || !(diff < INFINITY) || square == 0.0f) ? 0.0f : (den > 0.0f ? diff / den : INFINITY);
                            au_ratio = fmaxf(au_ratio, ratio);
                            au_outputs += 1;
                            au_listed += sure ? 0 : 1;
                            au_wrong += (sure && one != (yc > 0.0f)) ? 1 : 0;
                        }
                    }
                }
                if (__builtin_expect(__ballot(open) != 0, 0) && w0 + wi < n_words) {
                    const bool rows_differ = __builtin_amdgcn_readfirstlane(uneven[w]) != 0;
                    uint32_t which = 0;   // of the lane's outputs, 16 a tile
#pragma unroll
                    for (int t = 0; t < KT; ++t) {
                        uint32_t m = 0;
#pragma unroll
                        for (int v = 0; v < 16; ++v) m |= __builtin_fabsf(y[t][v]) >= bound[t] ? 0u : 1u << v;
                        if (bound[t] == INFINITY) m = 0xffffu;
                        if (rows_differ) {
                            m = 0;
#pragma unroll
                            for (int v = 0; v < 16; ++v) m |= sure_of(y[t][v], row_scale[w * 32 + v + 16 * half], xn[t]) ? 0u : 1u << v;
                        }
                        if (row + t * TK + c < a.n_rows) which |= m << (16 * t);
                    }
                    uint32_t both = code[0][wi] | (KT == 2 ? code[KT - 1][wi] << 16 : 0u);
                    while (__ballot(which != 0)) {
                        const int tv = which ? __builtin_ctz(which) : 0, v = tv % 16, bit = 31 - (v + 16 * half);
                        const int at_bit = tv - v + 15 - v;
                        const uint32_t behind = static_cast<uint32_t>(row - row0) + tv / 16 * TK + c;
                        const unsigned long long o = __ballot(which != 0);
                        if (listed <= kTilesList - 64) {
                            const int at = listed + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(o >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(o), 0u)));
                            // (with the bit as it will be stored)
                            if (which) list[at] = behind << 11 | ((both >> at_bit) & 1) << 10 | static_cast<uint32_t>(w) << 5 | static_cast<uint32_t>(bit);
                            listed += static_cast<int>(__builtin_popcountll(o));
                        } else if (which) {   // no room: at once (words that the list has open may not be stored yet)
                            float unused;
                            const uint32_t one = chain(row0 + behind, (31 - bit) * a.W + word0 + w, unused) > 0.0f;
                            both = (both & ~(1u << at_bit)) | one << at_bit;
                        }
                        which &= which - 1;
                    }
                    code[0][wi] = both & 0xffffu;
                    if constexpr (KT == 2) code[KT - 1][wi] = both >> 16;
                }
            }
            // ---- the words of a vector: 16 bits in either half of the wavefront
            uint32_t out[4];
#pragma unroll
            for (int wi = 0; wi < 4; ++wi) {
                if constexpr (KT == 2) {   // the lower half of the wavefront takes the first tile, the upper the second
                    const auto p = __builtin_amdgcn_permlane32_swap(code[0][wi], code[KT - 1][wi], false, false);
                    out[wi] = (p[0] << 16) | p[1];
                } else {
                    out[wi] = (code[0][wi] << 16) | other_half(code[0][wi]);
                }
            }
            const int64_t at = row + (KT == 2 ? half * TK : 0) + c;
            if (at < a.n_rows && (KT == 2 || half == 0)) {
                uint32_t* to = a.codes + xhead * a.code_head_stride + (a.code_row0 + at) * a.W + word0 + w0;
                if (a.W % 4 == 0) {
                    *reinterpret_cast<uint4*>(to) = make_uint4(out[0], out[1], out[2], out[3]);
                } else {
#pragma unroll
                    for (int wi = 0; wi < 4; ++wi)
                        if (w0 + wi < n_words) to[wi] = out[wi];
                }
            }
            if (listed > kTilesList / 2) settle_list();
        }
    }
    if (listed) settle_list();
    if constexpr (AUDIT) {
        const uint32_t outputs = wave_sum(au_outputs), listed_sum = wave_sum(au_listed), wrong = wave_sum(au_wrong);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) au_ratio = fmaxf(au_ratio, __shfl_xor(au_ratio, off));
        if (lane == 0) {
            atomicAdd(&a.audit->outputs, static_cast<unsigned long long>(outputs));
            if (listed_sum) atomicAdd(&a.audit->listed, static_cast<unsigned long long>(listed_sum));
            if (wrong) atomicAdd(&a.audit->wrong, static_cast<unsigned long long>(wrong));
            atomicMax(&a.audit->max_ratio_bits, __float_as_uint(au_ratio));   // non-negative floats order like their bits
        }
    }
}

// A workgroup takes a run of up to 16 tiles of one head (64, linear); the weights are fetched once per run.

// As many workgroups as runs of `run` tiles make, their runs as equal as they can be.
inline int even_runs(int64_t tiles, int run)
{
    const int64_t groups = (tiles + run - 1) / run;
    return static_cast<int>((tiles + groups - 1) / groups);
}

// The longest run, halved until the grid has `least` workgroups and no more than an eighth of their tiles is
// missing from the last ones.  512 heads x 600 binary32 vectors, 128 -> 128 -> 512, in runs of 16 and 3, 10 and 9, 4
// tiles: 1135, 710 and 752 us; x 90, in runs of 2 and 1, and of 1: 155 and 123 us.
inline int short_runs(int64_t tiles, int n_xheads, int least, int longest = 16)
{
    for (int run = longest; run > 1; run /= 2) {
        const int even = even_runs(tiles, run);
        const int64_t groups = (tiles + even - 1) / even;
        if (groups * n_xheads >= least && (groups * even - tiles) * 8 <= tiles) return even;
    }
    return 1;
}

// Workgroups on a compute unit at a time: `by_registers`, or what LDS holds.
inline int resident(const spotlight_ctx* ctx, int by_registers, size_t lds)
{
    int per_cu = by_registers;
    while (per_cu > 1 && per_cu * lds > static_cast<size_t>(ctx->max_lds)) --per_cu;
    return per_cu;
}

// The run for which the last generation of workgroups is not nearly empty: least is generations x (tiles +
// what the weights take, about a third of a tile).  The workgroups of a compute unit share its matrix cores:
// a last generation of no more than one for each counts two thirds.  8 heads, the longest run with 512 or
// 1024 workgroups and this one: 4000 / 8000 / 30000 vectors 128 -> 256 -> 128 60, 92, 299 and 51, 87, 276 us;
// 128 -> 512 -> 256 141, 266, 868 and 130, 233, 815 us; 128 -> 1024 -> 512 433, 846, 2922 and 395, 759, 2770 us.
inline int whole_generations(int64_t tiles, int n_xheads, int n_cus, int per_cu)
{
    const int64_t slots = static_cast<int64_t>(n_cus) * per_cu;
    int best = 1;
    int64_t best_cost = INT64_MAX;
    for (int run = 1; run <= 16; ++run) {
        const int64_t groups = (tiles + run - 1) / run * n_xheads, last = groups % slots;
        const int64_t thirds = groups / slots * 3 + (last == 0 ? 0 : last <= n_cus && per_cu > 1 ? 2 : 3);
        if (thirds * (3 * run + 1) < best_cost) {
            best = run;
            best_cost = thirds * (3 * run + 1);
        }
    }
    return even_runs(tiles, best);
}

// How the tiles of a head are shared out (share_of).
struct Shares {
    int parts, run, longer;
};
inline Shares equal_shares(int64_t tiles, int run) { return {static_cast<int>((tiles + run - 1) / run), run, 0}; }

// Whole generations, or where a compute unit has fewer tiles then, one generation whose runs differ by a tile:
// 4 heads x 313 tiles on 512 slots, runs of 3, six tiles on some compute units: 85.9 us; of 3 and 2, five: 78 us.
inline Shares shares_of(int64_t tiles, int n_xheads, int n_cus, int per_cu)
{
    const Shares even = equal_shares(tiles, whole_generations(tiles, n_xheads, n_cus, per_cu));
    const int64_t slots = static_cast<int64_t>(n_cus) * per_cu, parts = slots / n_xheads;
    if (parts < 1 || parts >= tiles || tiles / parts >= 16) return even;
    const int run = static_cast<int>(tiles / parts), longer = static_cast<int>(tiles % parts);
    // tiles of a compute unit, three times, and its weights
    const auto most = [&](int64_t groups) { return (groups + n_cus - 1) / n_cus; };
    const int64_t groups = static_cast<int64_t>(even.parts) * n_xheads, last = groups % slots;
    const int64_t cost_even = groups / slots * per_cu * (3 * even.run + 1) + most(last) * (3 * even.run + 1);
    const int64_t longs = static_cast<int64_t>(longer) * n_xheads;
    const int64_t cost = 3 * (static_cast<int64_t>(per_cu) * run + most(longs)) + per_cu;
    return cost < cost_even ? Shares{static_cast<int>(parts), run, longer} : even;
}

inline int launch_row_norms(spotlight_ctx* ctx, const HashArgs& a, int stage)
{
    constexpr int LPR = 16;
    const int n_out = a.n_wheads * a.L;
    StageTimer timer(ctx, stage, true);
    timer.launch(row_norm_kernel<LPR>, dim3(static_cast<unsigned>((n_out * LPR + kThreads - 1) / kThreads)), dim3(kThreads), 0, static_cast<const bf16_raw*>(a.w2), a.wnorm, n_out, a.hidden);
    return hip_rc(hipGetLastError());
}

template <typename XT, typename WT, int NW, int NUB, int NBW, bool AUDIT>
int launch(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage, size_t lds)
{
    auto kern = hash_bulk_kernel<XT, WT, NW, NUB, NBW, AUDIT>;
    if (allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kern), lds) != SPOTLIGHT_OK) return SPOTLIGHT_ERR_HIP;
    const int64_t tiles = (a.n_rows + kTile - 1) / kTile;
    // nothing is fetched once a run without a first layer or with weights read again for every tile (linear
    // binary32, 4 x 20000 vectors: 124 us with at least 4096 workgroups, 137 with 1024; 8 x 8000, binary32, 128 ->
    // 1024 -> 512: 959 us with short runs, 994 with whole generations); narrow layers have little to fetch, and more
    // workgroups share a compute unit
    constexpr int kShort = NUB == 0 ? 4096 : NUB < 0 || (NUB == 1 && NW == 4) ? 1024 : 0;
    const Shares shares = kShort ? equal_shares(tiles, short_runs(tiles, n_xheads, kShort))
                                 : shares_of(tiles, n_xheads, ctx->n_cus, resident(ctx, 4 * min_waves(NW, NBW) / NW, lds));
    if constexpr (NBW > 0) {
        if (const int rc = launch_row_norms(ctx, a, stage)) return rc;
    }
    dim3 grid(static_cast<unsigned>(shares.parts), static_cast<unsigned>(n_xheads));
    StageTimer timer(ctx, stage);
    timer.launch(kern, grid, dim3(NW * 64), lds, a, static_cast<float>(bulk_hash_eps(a.hidden, true)), shares.run, shares.longer);
    return hip_rc(hipGetLastError());
}

// LDS of hash_cert_kernel: what a tile takes, or the weights on their way into the registers
template <typename XT, int NW, int NUB>
size_t word_lds(const HashArgs& a)
{
    const size_t hp = hidden_padded(a.hidden);
    const size_t work = sizeof(float) * (XTile<XT>::kFloats + kTile * hs_stride(a.hidden) + hp) + hp * kTile * 2 * kept_operands<XT, NUB>() + sizeof(CertScratch<NW>);
    const size_t stage1 = static_cast<size_t>(a.hidden) * (kHeadDim * 2 + 16), stage2 = static_cast<size_t>(a.L) * (a.hidden * 2 + 16);
    return work > stage1 ? (work > stage2 ? work : stage2) : (stage1 > stage2 ? stage1 : stage2);
}

template <typename XT, int NW, int NUB, int WREG>
int launch_word(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage)
{
    const size_t lds = word_lds<XT, NW, NUB>(a);
    auto kern = hash_cert_kernel<XT, NW, NUB, WREG, false>;
    if (a.audit) kern = hash_cert_kernel<XT, NW, NUB, WREG, true>;
    if (allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kern), lds) != SPOTLIGHT_OK) return SPOTLIGHT_ERR_HIP;
    const int64_t tiles = (a.n_rows + kTile - 1) / kTile;
    // narrow layers have less to fetch per run, and more workgroups share a compute unit (8 x 65536, 128 -> 128
    // -> 64: 257 us with at least 2048, 267 with 1024)
    const Shares shares = NUB == 1 && NW == 4 ? equal_shares(tiles, short_runs(tiles, n_xheads, 2048)) : shares_of(tiles, n_xheads, ctx->n_cus, resident(ctx, 8 / NW, lds));
    dim3 grid(static_cast<unsigned>(shares.parts), static_cast<unsigned>(n_xheads));
    StageTimer timer(ctx, stage);
    timer.launch(kern, grid, dim3(NW * 64), lds, a, static_cast<float>(bulk_hash_eps(a.hidden, true)), shares.run, shares.longer);
    return hip_rc(hipGetLastError());
}

// Rounds a workgroup takes, one workgroup on a compute unit at a time: the fewest rounds in turn, the weights counted as one.
inline int rounds_of(int64_t all_rounds, int n_xheads, int n_cus)
{
    int64_t best = all_rounds, best_cost = INT64_MAX;
    const int64_t most = 4 * static_cast<int64_t>(n_cus) / n_xheads + 1;   // workgroups of a head
    for (int64_t groups = 1; groups <= most && groups <= all_rounds; ++groups) {
        const int64_t rounds = (all_rounds + groups - 1) / groups, used = (all_rounds + rounds - 1) / rounds;
        const int64_t cost = (used * n_xheads + n_cus - 1) / n_cus * (rounds + 1);
        if (cost < best_cost) { best = rounds; best_cost = cost; }
    }
    return static_cast<int>(best);
}

template <typename XT, int NB>
int launch_linear(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage)
{
    const size_t work = sizeof(LinearLds<XT>), staged = static_cast<size_t>(a.L < kLinearStage ? a.L : kLinearStage) * (kHeadDim * 2 + 16);
    const size_t lds = work > staged ? work : staged;
    auto kern = hash_linear_kernel<XT, NB, false>;
    if (a.audit) kern = hash_linear_kernel<XT, NB, true>;
    if (allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kern), lds) != SPOTLIGHT_OK) return SPOTLIGHT_ERR_HIP;
    const int64_t tiles = (a.n_rows + kTile - 1) / kTile;
    // a run of tiles pays for fetching R; the grid keeps two workgroups for every compute unit
    const int tpg = short_runs(tiles, n_xheads, 2 * ctx->n_cus, 64);
    dim3 grid(static_cast<unsigned>((tiles + tpg - 1) / tpg), static_cast<unsigned>(n_xheads));
    StageTimer timer(ctx, stage);
    timer.launch(kern, grid, dim3(kThreads), lds, a, static_cast<float>(bulk_hash_eps(kHeadDim, sizeof(XT) == 4)), tpg);
    return hip_rc(hipGetLastError());
}

template <typename XT>
int launch_linear_tiles(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage)
{
    const size_t lds = linear_lds(a.W < kLinearWords ? a.W : kLinearWords);
    auto kern = hash_linear_tiles_kernel<XT, false>;
    if (a.audit) kern = hash_linear_tiles_kernel<XT, true>;
    if (allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kern), lds) != SPOTLIGHT_OK) return SPOTLIGHT_ERR_HIP;
    const int per_round = kTile * (sizeof(XT) == 2 ? 2 : 1) * kLinearWaves;
    const int64_t all_rounds = (a.n_rows + per_round - 1) / per_round;
    const int groups = (a.W + kLinearWords - 1) / kLinearWords;
    const int most = (1 << 21) / per_round;   // rows in a list entry
    const int rounds = std::min(rounds_of(all_rounds, n_xheads * groups, ctx->n_cus), most);
    dim3 grid(static_cast<unsigned>((all_rounds + rounds - 1) / rounds), static_cast<unsigned>(n_xheads), static_cast<unsigned>(groups));
    StageTimer timer(ctx, stage);
    timer.launch(kern, grid, dim3(kLinearWaves * 64), lds, a, rounds);
    return hip_rc(hipGetLastError());
}

template <typename XT, int NW, int NUB, int NBW>
int launch_cert(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage, size_t lds)
{
    if (a.audit) return launch<XT, bf16_raw, NW, NUB, NBW, true>(ctx, a, n_xheads, stage, lds);
    return launch<XT, bf16_raw, NW, NUB, NBW, false>(ctx, a, n_xheads, stage, lds);
}

// Workgroups that share a segment of open rows: the chip is filled, and not by a last generation that is nearly empty;
// each fetches the weights (a thirtieth of a segment's tiles).
inline int open_parts(int64_t segments, int slots)
{
    int best = 1;
    double best_cost = 1e30;
    for (int parts = 1; parts <= slots; ++parts) {
        const double cost = static_cast<double>((segments * parts + slots - 1) / slots) * (1.0 / parts + 0.03);
        if (cost < best_cost) { best = parts; best_cost = cost; }
    }
    return best;
}

// The grid of a second pass on a chip that holds `slots` of its workgroups, and its kernels' `run` (open_job).  By what is open where every
// segment can have two workgroups and more.
struct OpenGrid {
    dim3 grid;
    int run;
};
inline OpenGrid open_grid(const HashArgs& a, int n_xheads, int slots)
{
    const int64_t segments = segments_of(a), all = segments * n_xheads;
    if (a.open_counts && 2 * all <= slots) return {dim3(static_cast<unsigned>(slots)), -n_xheads};
    const int parts = open_parts(all, slots);
    return {dim3(static_cast<unsigned>(segments * parts), static_cast<unsigned>(n_xheads)), parts};
}

inline size_t align16(size_t bytes) { return (bytes + 15) / 16 * 16; }

template <int NW, int NUB, int NBW>
int launch_open(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage, size_t work)
{
    using T = bf16_raw;
    const size_t open_at = align16(work), lds = open_at + sizeof(OpenRows);
    auto kern = hash_bulk_kernel<T, T, NW, NUB, NBW, false, true>;
    if (allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kern), lds) != SPOTLIGHT_OK) return SPOTLIGHT_ERR_HIP;
    const OpenGrid g = open_grid(a, n_xheads, ctx->n_cus * resident(ctx, 4 * min_waves(NW, NBW) / NW, lds));
    if (const int rc = launch_row_norms(ctx, a, stage)) return rc;
    StageTimer timer(ctx, stage);
    timer.launch(kern, g.grid, dim3(NW * 64), lds, a, static_cast<float>(bulk_hash_eps(a.hidden, true)), g.run, static_cast<int>(open_at));
    return hip_rc(hipGetLastError());
}

template <int NW, int NUB, int WREG>
int launch_word_open(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage)
{
    using T = bf16_raw;
    const size_t open_at = align16(word_lds<T, NW, NUB>(a)), lds = open_at + sizeof(OpenRows);
    auto kern = hash_cert_kernel<T, NW, NUB, WREG, false, true>;
    if (allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kern), lds) != SPOTLIGHT_OK) return SPOTLIGHT_ERR_HIP;
    // narrow layers leave room for a third workgroup: 8 heads x 65536 keys, all open, 128 -> 64 -> 64 646 us with two, 470 with three, 128 -> 128 -> 64 940 and
    // 770; random keys 20 and 19, 32 and 27.  More segments than are shared out by their open rows have few tiles each: 512 heads x 257, 128 -> 64 -> 32, the call 39 and 47
    const OpenGrid g = open_grid(a, n_xheads, ctx->n_cus * resident(ctx, NUB == 1 && a.open_counts ? 3 : 2, lds));
    StageTimer timer(ctx, stage);
    timer.launch(kern, g.grid, dim3(NW * 64), lds, a, static_cast<float>(bulk_hash_eps(a.hidden, true)), g.run, static_cast<int>(open_at));
    return hip_rc(hipGetLastError());
}

// Which of the two kernels of the linear hash: with a tile or two for a wavefront, the one that spreads the words of a tile over
// its wavefronts is done sooner; longer codes need fewer tiles to fill the other's time, short ranges of a head leave
// its workgroups half empty.  That one and the other, bfloat16: 32 bits, 32000 and 65536 vectors 11.6, 17.1 and 12.4,
// 12.4 us; 128 bits, 20000 and 32000 10.1, 15.7 and 13.3, 13.0; 512 bits, 4800 and 19200 20.8, 49.2 and 25.3, 26.1;
// 1024 bits, 32 22.9 and 17.6; 512 heads x 100, 32 and 512 bits 15.5, 52.4 and 17.1, 40.1; x 32, 512 bits 30.2 and 37.0.
inline bool linear_by_tiles(const spotlight_ctx* ctx, const HashArgs& a, int n_xheads)
{
    const int64_t tiles = (a.n_rows + kTile - 1) / kTile * n_xheads;
    const int fill = a.W == 1 ? 8 : a.W < 16 ? 4 : 1;
    return a.W > kLinearWords || tiles >= fill * (a.n_rows < 256 ? 3 : 1) * static_cast<int64_t>(ctx->n_cus);
}

inline size_t lds_bytes(size_t x_size, int hidden) { return kTile * (x_size * kHeadDim + sizeof(float) * static_cast<size_t>(hidden_padded(hidden))); }

}  // namespace bulk

// Whether the matrix-core kernels serve this job: enough vectors, and the activations of a tile fit in
// LDS (hidden widths up to 1152, or 1216 with bfloat16 vectors).
inline bool bulk_hash_applies(const spotlight_ctx* ctx, const hashdev::HashArgs& a, int n_xheads, size_t x_size, size_t w_size)
{
    // From how many vectors per head: below, the vector-ALU kernel's tiles of 8 do less work for padding.
    // Measured for 8 / 512 heads of a 128 -> 256 -> 128 network: 8 rows 26 against 23 and 28 against 31 us,
    // 9 rows 26 against 23 and 34 against 31 us, 17 rows 26 against 23 and 48 against 32 us; 128 -> 512 -> 256:
    // 9 rows 53 against 48 and 70 against 75 us; linear, 512 bits: 31 rows 19 against 20 us, 100 rows 40 against 20 us.
    const int min_rows = a.hidden == 0 ? bulk::kTile : n_xheads > ctx->n_cus ? 17 : 9;
    // Codes of one or two words with a wide hidden layer: while every tile of 8 has a compute unit of its own
    // that kernel is the faster one, its lanes sharing the sums.  8 heads x 20 vectors, 64 bits: hidden 256 19.2
    // against 22.1 us, 512 34 against 46 us; hidden 128 17 against 14 us; 512 heads x 18, 256 -> 64: 45 against 31 us.
    const bool few = a.n_rows < bulk::kTile && n_xheads * ((a.n_rows + 7) / 8) <= ctx->n_cus;
    if (few && a.hidden > 128 && a.W <= 2) return false;
    // Likewise long codes behind a narrow layer of binary32 weights, whose words a wavefront takes one after another.
    // 8 heads x 17: 128 -> 64 -> 512 18.2 against 19.5 us, 1024 bits 25.7 against 31; 384 bits 18.4 against 16.3.
    if (few && w_size == 4 && a.hidden <= 128 && a.W >= 16) return false;
    // One word of bfloat16 weights has one wavefront of eight or sixteen at work in layer 2: up to three tiles of 8 are
    // the faster ones on any grid.  512 heads x 17, 32 bits: hidden 512 68 against 73 us, 1024 172 against 184;
    // hidden 256 40 against 28; binary32 weights 100 against 73.
    if (w_size == 2 && a.hidden > 256 && a.hidden <= 1024 && a.W == 1 && a.n_rows <= 24) return false;
    // Exact words, one or more for every hidden unit, on grids of more than two tiles for every compute unit: their
    // loads and signs are all there is, and the vector-ALU kernel spreads those over all its lanes.  512 heads x 600,
    // 128 -> 16 -> 1024: 345 against 500 us; 512 bits, binary32 249 against 298; 256 bits 206 against 202; 8 heads x
    // 300, 1024 bits 39 against 21.
    const bool exact = w_size == 4 || a.hidden % 16 != 0 || a.W > 16;
    if (exact && a.hidden > 0 && a.W >= a.hidden && (a.n_rows + bulk::kTile - 1) / bulk::kTile * n_xheads > 2 * ctx->n_cus) return false;
    return a.wnorm && a.n_rows >= min_rows && bulk::lds_bytes(x_size, a.hidden) <= static_cast<size_t>(ctx->max_lds);
}

// The rows a first pass left open (a.open), with the chain: bfloat16 vectors and weights, hidden a multiple of 16
// up to 1024, codes up to 256 bits.
inline int run_open_hash(spotlight_ctx* ctx, const hashdev::HashArgs& a, int n_xheads, int stage)
{
    using namespace bulk;
    const size_t lds = lds_bytes(2, a.hidden);
    const int nub = hidden_padded(a.hidden) / 32;
    if (a.W <= 4 && nub <= 4) return launch_word_open<4, 1, 8>(ctx, a, n_xheads, stage);
    if (a.W <= 4 && nub <= 8) return launch_word_open<4, 2, 16>(ctx, a, n_xheads, stage);
    if (nub <= 4) return launch_open<4, 1, 2>(ctx, a, n_xheads, stage, lds);
    if (nub <= 8) return launch_open<4, 2, 2>(ctx, a, n_xheads, stage, lds);
    if (nub <= 16) return launch_open<8, 2, 1>(ctx, a, n_xheads, stage, lds);
    return launch_open<16, 2, 1>(ctx, a, n_xheads, stage, lds);
}

// Bulk hashing in two passes (hash_screen.h); declared here for the dispatch in hash.hip.
bool screened_hash_applies(const spotlight_ctx* ctx, const hashdev::HashArgs& a, int n_xheads);
int run_screened_hash(spotlight_ctx* ctx, const hashdev::HashArgs& a, int n_xheads, int stage);

template <typename XT, typename WT>
int run_bulk_hash(spotlight_ctx* ctx, const hashdev::HashArgs& a, int n_xheads, int stage)
{
    using namespace bulk;
    const size_t lds = lds_bytes(sizeof(XT), a.hidden);
    const int nub = hidden_padded(a.hidden) / 32;
    const int64_t tiles = (a.n_rows + kTile - 1) / kTile * n_xheads;
    if constexpr (sizeof(WT) == 2) {
        if (nub == 0) {
            if (linear_by_tiles(ctx, a, n_xheads)) return launch_linear_tiles<XT>(ctx, a, n_xheads, stage);
            if (a.W <= 4) return launch_linear<XT, 1>(ctx, a, n_xheads, stage);
            if (a.W <= 8) return launch_linear<XT, 2>(ctx, a, n_xheads, stage);
            return launch_linear<XT, 4>(ctx, a, n_xheads, stage);
        }
        if (a.hidden % 16 == 0 && a.W <= 4 && nub <= 4) return launch_word<XT, 4, 1, 8>(ctx, a, n_xheads, stage);
        // Where no compute unit gets a second tile, a block of hidden units for each of eight wavefronts: the tile is done
        // sooner, and no other workgroup would hide the waits of four.  One pass over 1 to 256 tiles, 128 -> 256 ->
        // 128 23 and 18 us, 160 -> 64 15 - 18 and 13 - 15; 512 tiles 29 and 34.
        if (a.hidden % 16 == 0 && a.W <= 4 && nub > 4 && nub <= 8)
            return tiles <= ctx->n_cus ? launch_word<XT, 8, 1, 16>(ctx, a, n_xheads, stage) : launch_word<XT, 4, 2, 16>(ctx, a, n_xheads, stage);
        if (a.hidden % 16 == 0 && a.W <= 16 && nub <= 32) {
            if (nub <= 4) {
                if (a.W <= 8) return launch_cert<XT, 4, 1, 2>(ctx, a, n_xheads, stage, lds);
                return launch_cert<XT, 4, 1, 4>(ctx, a, n_xheads, stage, lds);
            }
            if (nub <= 8) {
                if (a.W <= 8) return launch_cert<XT, 4, 2, 2>(ctx, a, n_xheads, stage, lds);
                return launch_cert<XT, 4, 2, 4>(ctx, a, n_xheads, stage, lds);
            }
            // wide hidden layers: eight wavefronts, because LDS holds only one or two workgroups
            if (nub <= 16) {
                if (a.W <= 8) return launch_cert<XT, 8, 2, 1>(ctx, a, n_xheads, stage, lds);
                return launch_cert<XT, 8, 2, 2>(ctx, a, n_xheads, stage, lds);
            }
            return launch_cert<XT, 16, 2, 1>(ctx, a, n_xheads, stage, lds);
        }
    }
    if constexpr (sizeof(WT) == 4) {
        if (nub == 0) return launch<XT, WT, 4, 0, 0, false>(ctx, a, n_xheads, stage, lds);
    }
    if (nub <= 4) return launch<XT, WT, 4, 1, 0, false>(ctx, a, n_xheads, stage, lds);
    // Eight wavefronts where four have more than a code word each, and where no compute unit gets a second tile:
    // the tile is done sooner (8 heads x 20 binary32 vectors, 128 -> 256 -> 256: 25.6 against 30.8 us; 128 bits:
    // 21.2 against 22.8; 8 x 65536, 256 bits: 1251 against 1276).  Otherwise the four hide each other's waits
    // better (4 x 4 x 10000, 32 bits: 276 against 304 us).
    if (nub > 4 && nub <= 8 && (a.W > 4 || tiles <= ctx->n_cus)) return launch<XT, WT, 8, 1, 0, false>(ctx, a, n_xheads, stage, lds);
    if (nub <= 8) return launch<XT, WT, 4, 2, 0, false>(ctx, a, n_xheads, stage, lds);
    if (nub <= 16) return launch<XT, WT, 8, 2, 0, false>(ctx, a, n_xheads, stage, lds);
    return launch<XT, WT, 8, -1, 0, false>(ctx, a, n_xheads, stage, lds);
}

}  // namespace spotlight
