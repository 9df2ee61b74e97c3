// Bulk hashing, second pass, for hidden layers of 272 to 512 units and codes of 160 to 256 bits: the keys that the first pass
// (hash_screen.h) left open.
//
// The same work as hash_cert_kernel: layer 1 with the chain on the binary32 matrix instruction, layer 2 on the
// bfloat16 one with the bound, what that leaves open with the chain.  Eight wavefronts, one workgroup on a compute unit
// (its LDS holds the activations three times, as there: 154 KB at 512 units).  The weights of layer 1 stay in registers, those of layer 2
// come from the first pass's copy, in operand order, eight steps ahead: hash_bulk_kernel, which this replaces, read
// them a row per lane a step ahead, split all activations in every wavefront, and waited two thirds of its time.
// Rows = the outputs of a word and columns = keys, as in the first pass, so that a lane has the signs of one key.  Half of the
// open keys still have an output within this bound: those of a tile go to a list, and one wavefront in turn runs their chains, a
// lane each, while the others are at layer 1 of the next tile (every wavefront its own: half of all vector instructions).
// 8 heads x 131072 keys, 128 -> 512 -> 256, 27 % open: 985 and 890 us; x 16384 171 and 126 us; 128 -> 288 -> 256 1.1x.
// Left out in turn (timing only): layer 1 292 us, layer 2 240 (its weights are 256 KB of L2 a tile), the chains 177, SiLU 104.
// Half of layer 2's weights in registers as well: 51 - 61 spilled, 940 us.
#pragma once
#include "hash_screen.h"

namespace spotlight {
namespace screen {

constexpr int kOpenWaves = 8;         // each has two blocks of hidden units and a code word

__host__ __device__ constexpr int open_stride(int hidden) { return blocks_of(hidden) * 32 + 4; }   // words a key: b128 accesses of 8 lanes miss each other
constexpr int kChains = 512;          // open outputs of a tile that go to its list
// Wavefronts that run the chains of a tile's list of n.
__host__ __device__ constexpr int chain_waves(int n) { return n <= 64 ? 1 : kOpenWaves; }
struct OpenScratch {
    float part[kOpenWaves][bulk::kTile];   // sums of squares of the wavefronts' activations
    uint32_t codes[kOpenWaves][bulk::kTile];
    uint16_t list[kChains];                // key | word << 5 | output in the order of its bits << 8
    uint32_t listed[2];                    // of a tile and the next
};
inline size_t open_lds(int hidden)
{
    const size_t hp = static_cast<size_t>(blocks_of(hidden)) * 32;
    return bulk::align16(sizeof(float) * (2 * bulk::XTile<bf16_raw>::kFloats + bulk::kTile * open_stride(hidden) + hp) + hp * bulk::kTile * 4 + sizeof(OpenScratch));
}

// WM: code words the first pass laid the operands out for.
template <int WM, typename Record>
__global__ __launch_bounds__(kOpenWaves * 64, 2) void hash_open_kernel(HashArgs a, const char* __restrict__ scales, const uint4* __restrict__ operands, int run, int open_at, Record record)
{
    constexpr int TK = bulk::kTile, NT = kOpenWaves * 64, NUB = 2, OPS = operands_of(WM);
    using bulk::XTile;
    extern __shared__ __align__(16) float lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, half = lane >> 5;
    bulk::OpenRows& list = *reinterpret_cast<bulk::OpenRows*>(reinterpret_cast<char*>(lds) + open_at);
    const bulk::OpenJob job = bulk::open_job(list, a, run, wave, lane);
    if (job.parts == 0) return;
    const int xhead = job.xhead;
    const int whead = whead_of(a, xhead);
    const int nub = blocks_of(a.hidden), stride = open_stride(a.hidden), W = a.W;
    float* xs = lds;                                                        // the x tile and the next one
    float* hs = xs + 2 * XTile<bf16_raw>::kFloats;                          // [TK][stride]
    uint4* hilo = reinterpret_cast<uint4*>(hs + TK * stride);               // [2 nub steps of 16 units][hi, lo][64]
    float* bias = reinterpret_cast<float*>(hilo + nub * 2 * 2 * 64);        // [blocks][32]
    OpenScratch& m = *reinterpret_cast<OpenScratch*>(bias + nub * 32);

    const int64_t first = job.first;
    bulk::OpenWalk walk{list, a.open + xhead * a.open_stride + first,
                        static_cast<int>(min(a.n_rows - first * TK, static_cast<int64_t>(bulk::kOpenSegment))), 0, 0, 0, 0, 0};
    if (!walk.begin(job.part, job.parts, tid, NT) || !walk.advance(wave, lane)) return;

    const bf16_raw* b1 = static_cast<const bf16_raw*>(a.b1) + static_cast<int64_t>(whead) * a.hidden;
    const bf16_raw* w2 = static_cast<const bf16_raw*>(a.w2) + static_cast<int64_t>(whead) * a.L * a.hidden;
    const WordScale* ws = reinterpret_cast<const WordScale*>(scales + static_cast<int64_t>(whead) * (1 + W) * 16) + 1;
    const uint4* from = operands + static_cast<int64_t>(whead) * nub * OPS * 64 + lane;
    const int word = min(wave, W - 1);                               // wavefronts without one have layer 1 only
    const float scale = ws[word].s2;
    const uint32_t zeros = ws[word].zeros;
    const bool uneven = ws[word].uneven != 0;
    const RowScale* rows_of_word = row_scales(scales, a.n_wheads, whead, W) + word * 32 + 16 * half;
    const int n_mine = max(0, min(NUB, nub - wave * NUB));           // blocks of this wavefront

    bulk::UnitBlock<bf16_raw> ublk[NUB];                             // layer 1: the operands of the 64 steps
#pragma unroll
    for (int i = 0; i < NUB; ++i) {
        if (i >= n_mine) continue;
#pragma unroll
        for (int g = 0; g < 8; ++g) {   // k = 16 g .. + 7 in the lower half, 16 g + 8 .. + 15 in the upper
            const uint4 w = from[((wave * NUB + i) * OPS + g) * 64];
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
    constexpr int PF = 8;            // steps of layer 2 whose weights are on their way
    const int n_ks = 2 * nub;
    auto weights = [&](int ks) { return from[((ks / 2) * OPS + 8 + (ks % 2) * WM + word) * 64]; };
    for (int i = tid; i < nub * 32; i += NT) bias[i] = i < a.hidden ? load1(b1 + i) : 0.0f;

    // the x tile, fetched ahead: thread e has 8 elements of vector e % 32
    Raw8<bf16_raw> xr;
    const bf16_raw* xhead_base = static_cast<const bf16_raw*>(a.x) + xhead * a.x_head_stride + a.x_row0 * kHeadDim;
    auto row_of = [&](int item) { return first * TK + walk.list.row[item]; };
    auto fetch_x = [&](int tile) { load_raw(xhead_base + row_of(min(tile * TK + tid % TK, walk.count - 1)) * kHeadDim + (tid / TK) * 8, xr); };   // past the end: a stand-in
    auto put_x = [&](int buf) { XTile<bf16_raw>::put(xs + buf * XTile<bf16_raw>::kFloats, tid / TK, tid % TK, xr); };

    // the chain of output row j for key t of the tile, whose activations are in LDS
    auto chain = [&](int j, int t) {
        constexpr int PF = 16;   // groups of 8 weights on their way
        const bf16_raw* row = w2 + static_cast<int64_t>(j) * a.hidden;
        const float* hr = hs + t * stride;
        const int n8 = a.hidden / 8;
        float y = 0.0f;
        Raw8<bf16_raw> ahead[PF];
#pragma unroll
        for (int p = 0; p < PF; ++p) load_raw(row + 8 * min(p, n8 - 1), ahead[p]);
#pragma unroll 1
        for (int g0 = 0; g0 < n8; g0 += PF) {
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                if (g0 + p < n8) {
                    float wv[8];
                    expand(ahead[p], wv);
                    load_raw(row + 8 * min(g0 + PF + p, n8 - 1), ahead[p]);
                    const float4 f0 = *reinterpret_cast<const float4*>(hr + (g0 + p) * 8), f1 = *reinterpret_cast<const float4*>(hr + (g0 + p) * 8 + 4);
                    const float hv[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e) y = __builtin_fmaf(wv[e], hv[e], y);
                }
            }
        }
        return y;
    };

    auto settle = [&](int t, int w, int out) {
        const uint32_t bit = 1u << (31 - out);
        if (((m.codes[w][t] & bit) != 0) != (chain(out * W + w, t) > 0.0f)) atomicXor(&m.codes[w][t], bit);
    };
    if (tid < 2) m.listed[tid] = 0;
    fetch_x(0);
    int turn = 0;                    // tiles so far
    bool more = true;
    while (more) {
        put_x(0);
        __syncthreads();
        for (int tile = 0; tile < walk.tiles; ++tile, ++turn) {
            const int buf = tile & 1;
            if (tile + 1 < walk.tiles) fetch_x(tile + 1);   // in flight during layer 1

            // ---- layer 1, while other wavefronts may still be at the previous tile's chains
            f32x16_t h[NUB];
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
                for (int s = 0; s < kHeadDim / 2; ++s)
                    h[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(ublk[i].step(s), XTile<bf16_raw>::step(xs + buf * XTile<bf16_raw>::kFloats, s, lane), h[i], 0, 0, 0);
            }
            __syncthreads();   // the previous tile's activations are no longer needed, nor its number of chains
            if (tid == 0) m.listed[~turn & 1] = 0;
            if (tile + 1 < walk.tiles) put_x(buf ^ 1);
            // layer 2's first weights, in flight meanwhile
            uint4 ahead[PF];
#pragma unroll
            for (int p = 0; p < PF; ++p) ahead[p] = weights(min(p, n_ks - 1));
            float sumsq = 0.0f;
#pragma unroll
            for (int i = 0; i < NUB; ++i) {
                if (i >= n_mine) continue;
                const int ub = wave * NUB + i;
#pragma unroll
                for (int j = 0; j < 2; ++j) {   // accumulators 8 j .. 8 j + 7: units 16 j + 8 half .. + 7 of the block
                    float h8[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        h8[e] = silu(h[i][8 * j + e]);
                        sumsq = __builtin_fmaf(h8[e], h8[e], sumsq);
                        if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // four at a time: more side by side would spill
                    }
                    float4* f = reinterpret_cast<float4*>(hs + c * stride + ub * 32 + 16 * j + 8 * half);
                    f[0] = make_float4(h8[0], h8[1], h8[2], h8[3]);
                    f[1] = make_float4(h8[4], h8[5], h8[6], h8[7]);
                    bf16x8_t hi, lo;
                    bulk::split8(h8, hi, lo);
                    hilo[((ub * 2 + j) * 2 + 0) * 64 + lane] = __builtin_bit_cast(uint4, hi);
                    hilo[((ub * 2 + j) * 2 + 1) * 64 + lane] = __builtin_bit_cast(uint4, lo);
                }
            }
            sumsq = add_halves(sumsq);
            if (half == 0) m.part[wave][c] = sumsq;
            __syncthreads();   // activations and norms are complete, and the next x tile

            // ---- layer 2 of this wavefront's word
            if (wave < W) {
                float square = 0.0f;
#pragma unroll
                for (int p = 0; p < kOpenWaves; ++p) square += m.part[p][c];
                const float hn = 1.001f * __builtin_amdgcn_sqrtf(square) + kSlack;
                f32x16_t y;
#pragma unroll
                for (int v = 0; v < 16; ++v) y[v] = 0.0f;
                if (zeros) {   // rows of zeros: far from zero, and negative
#pragma unroll
                    for (int v = 0; v < 16; ++v) y[v] = (zeros >> (v + 16 * half)) & 1 ? -1e30f : 0.0f;
                }
#pragma unroll 1
                for (int ks0 = 0; ks0 < n_ks; ks0 += PF) {
#pragma unroll
                    for (int p = 0; p < PF; ++p) {
                        const int ks = ks0 + p;
                        if (ks >= n_ks) continue;
                        const bf16x8_t b = __builtin_bit_cast(bf16x8_t, ahead[p]);
                        ahead[p] = weights(min(ks + PF, n_ks - 1));
                        y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, __builtin_bit_cast(bf16x8_t, hilo[(ks * 2 + 0) * 64 + lane]), y, 0, 0, 0);
                        y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, __builtin_bit_cast(bf16x8_t, hilo[(ks * 2 + 1) * 64 + lane]), y, 0, 0, 0);
                    }
                }
                // ---- signs, and which outputs are too close to zero to trust
                float bound = 1.002f * (scale * hn);
                if (!(bound < 1e25f)) bound = INFINITY;   // also where it is no number
                auto own_bound = [&](int v) { return 1.002f * (rows_of_word[v].s2 * hn); };
                if (tile * TK + c < walk.count) record(xhead, row_of(tile * TK + c), wave, half, y, [&](int v) { return uneven ? own_bound(v) : bound; });
                uint32_t sign = 0, which = 0;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    sign = __builtin_amdgcn_alignbit(sign, __float_as_uint(y[v]), 31);
                    which |= __builtin_fabsf(y[v]) >= bound ? 0u : 1u << v;
                }
                if (bound == INFINITY) which = 0xffffu;
                if (uneven) {   // each output and the bound of its own row
                    which = 0;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float b = own_bound(v);
                        which |= __builtin_fabsf(y[v]) >= b && b < 1e25f ? 0u : 1u << v;
                        if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (tile * TK + c >= walk.count) which = 0;   // a stand-in
                uint32_t code = ~sign & 0xffffu;
                code = (code << 16) | other_half(code);
                if (half == 0) m.codes[wave][c] = code;
                while (__ballot(which != 0)) {   // every lane's next open output, to the list; no room: at once
                    const unsigned long long o = __ballot(which != 0);
                    uint32_t at = 0;
                    if (lane == 0) at = atomicAdd(&m.listed[turn & 1], static_cast<uint32_t>(__builtin_popcountll(o)));
                    at = __builtin_amdgcn_readfirstlane(at) + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(o >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(o), 0u));
                    if (which) {
                        const int out = __builtin_ctz(which) + 16 * half;
                        which &= which - 1;
                        if (at < static_cast<uint32_t>(kChains)) m.list[at] = static_cast<uint16_t>(c | word << 5 | out << 8);
                        else settle(c, word, out);
                    }
                }
            }
            __syncthreads();   // the tile's codes and list are complete
            // ---- one wavefront runs the chains, a lane each, and stores the codes; the others are at the next tile's layer 1.  More than
            // a lane can have at once are shared by all: every key with 16 (4) open outputs, 8 x 32768, 2460 (1320) us by one wavefront, 1270 (1000) by all.
            const int n = __builtin_amdgcn_readfirstlane(min(static_cast<int>(m.listed[turn & 1]), kChains));
            const int sharers = chain_waves(n);
            if (sharers > 1) {
                for (int e = tid; e < n; e += NT) settle(m.list[e] & 31, (m.list[e] >> 5) & 7, m.list[e] >> 8);
                __syncthreads();
            }
            if (wave == turn % kOpenWaves) {
                if (sharers == 1) {
                    for (int e = lane; e < n; e += 64) settle(m.list[e] & 31, (m.list[e] >> 5) & 7, m.list[e] >> 8);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                }
                const int rows = min(TK, walk.count - tile * TK);
                for (int e = lane; e < rows * W; e += 64)
                    a.codes[xhead * a.code_head_stride + (a.code_row0 + row_of(tile * TK + e / W)) * W + e % W] = m.codes[e % W][e / W];
            }
        }
        more = walk.advance(wave, lane);
        if (more) fetch_x(0);
    }
}

// Whether this kernel serves the second pass of a network.
inline bool open_serves(int hidden, int W) { return hidden > 256 && hidden <= 512 && words_for(W) == 8 && !resident(hidden, W); }

template <typename Record = NoRecord>
int launch_open(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage, Record record = {})
{
    const size_t open_at = open_lds(a.hidden), lds = open_at + sizeof(bulk::OpenRows);
    auto kern = hash_open_kernel<8, Record>;
    if (allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kern), lds) != SPOTLIGHT_OK) return SPOTLIGHT_ERR_HIP;
    const bulk::OpenGrid g = bulk::open_grid(a, n_xheads, ctx->n_cus);
    StageTimer timer(ctx, stage);
    timer.launch(kern, g.grid, dim3(kOpenWaves * 64), lds, a, static_cast<const char*>(a.scales), static_cast<const uint4*>(a.operands), g.run, static_cast<int>(open_at), record);
    return hip_rc(hipGetLastError());
}

}  // namespace screen
}  // namespace spotlight
