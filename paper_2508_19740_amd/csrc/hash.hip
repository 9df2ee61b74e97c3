// Hash MLP + sign + bit-packing (paper Sec. 3.2 Eq. 4-6, appendix "Bit-Packing CUDA Kernel").
//
// One workgroup hashes a tile of TK vectors of one head.  Every output keeps its own binary32
// accumulator and takes its fused multiply-adds in increasing index order, so the sign bits do not
// depend on the tile size or launch shape:
//   a_i = b1_i + sum_k W1[i][k] x[k];  h_i = a_i / (1 + exp(-a_i));  y_j = sum_i W2[j][i] h_i
// exp is the fixed routine silu_exp() (range clamp, round-to-nearest reduction by ln 2 in two fused
// steps, degree-7 Horner polynomial, exact power-of-two scaling).
//
// Phase 1: thread i owns hidden unit i (+256, ...), streams its W1 row from global memory 8 values
//          at a time and reads x from LDS (stored [k][t], so one 16-byte LDS read feeds 4 vectors).
// Phase 2: a wavefront owns two code words; lane l computes the hash output that belongs to bit
//          (l & 31) of word 2p + (l >> 5), i.e. output (31 - (l & 31)) * W + word, so a wave-wide
//          ballot of (y > 0) IS the pair of packed words.  No boolean tensor is ever stored.
#include "hash_bulk.h"
#include "hash_vec.h"

namespace spotlight {
using namespace hashdev;
extern template int run_bulk_hash<float, float>(spotlight_ctx*, const HashArgs&, int, int);
extern template int run_bulk_hash<float, bf16_raw>(spotlight_ctx*, const HashArgs&, int, int);
extern template int run_bulk_hash<bf16_raw, float>(spotlight_ctx*, const HashArgs&, int, int);
extern template int run_bulk_hash<bf16_raw, bf16_raw>(spotlight_ctx*, const HashArgs&, int, int);
namespace {

// TK consecutive floats from LDS (16-byte reads when TK is a multiple of 4)
template <int TK>
__device__ __forceinline__ void lds_tile(const float* p, float (&o)[TK])
{
    if constexpr (TK % 4 == 0) {
#pragma unroll
        for (int t = 0; t < TK / 4; ++t) {
            const float4 v = reinterpret_cast<const float4*>(p)[t];
            o[4 * t] = v.x; o[4 * t + 1] = v.y; o[4 * t + 2] = v.z; o[4 * t + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int t = 0; t < TK; ++t) o[t] = p[t];
    }
}

// acc[t] += sum over n8*8 consecutive weights of `row` times act[(i)*stride + t], in increasing i,
// one fused multiply-add per term.  PF groups of 8 weights are fetched ahead of their use.
template <typename WT, int TK, int PF>
__device__ __forceinline__ void dot_rows(const WT* __restrict__ row, int n8, const float* act, int stride,
                                         float (&acc)[TK])
{
    int g = 0;
    for (; g + PF <= n8; g += PF) {
        float wv[PF][8];
#pragma unroll
        for (int p = 0; p < PF; ++p) load8(row + (g + p) * 8, wv[p]);
#pragma unroll
        for (int p = 0; p < PF; ++p)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float xr[TK];
                lds_tile<TK>(act + ((g + p) * 8 + j) * stride, xr);
#pragma unroll
                for (int t = 0; t < TK; ++t) acc[t] = __builtin_fmaf(wv[p][j], xr[t], acc[t]);
            }
    }
    for (; g < n8; ++g) {
        float wv[8];
        load8(row + g * 8, wv);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float xr[TK];
            lds_tile<TK>(act + (g * 8 + j) * stride, xr);
#pragma unroll
            for (int t = 0; t < TK; ++t) acc[t] = __builtin_fmaf(wv[j], xr[t], acc[t]);
        }
    }
}

// LDS: xs [128][TK] floats, then hs [hidden][TK] floats (hidden > 0 only).
template <typename XT, typename WT, int TK, int KSPLIT>
__global__ __launch_bounds__(kThreads) void hash_kernel(HashArgs a)
{
    constexpr int TK2 = TK / KSPLIT;
    constexpr int PF = TK == 1 ? 16 : (TK <= 8 ? 2 : 1);  // weight groups fetched ahead
    extern __shared__ __align__(16) float lds[];
    float* xs = lds;
    float* hs = lds + kHeadDim * TK;

    const int tid = threadIdx.x;
    const int xhead = blockIdx.y;
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * TK;
    const int rows = static_cast<int>(min(static_cast<int64_t>(TK), a.n_rows - r0));
    const int whead = (xhead % a.heads_per_batch) / a.group;
    if (a.zero && blockIdx.x == 0)
        for (int i = tid; i < a.zero_words; i += kThreads) a.zero[static_cast<int64_t>(xhead) * a.zero_words + i] = 0u;

    // ---- stage the x tile, transposed to [k][t], rows past the end as zeros
    const XT* xbase = static_cast<const XT*>(a.x) + xhead * a.x_head_stride + (a.x_row0 + r0) * kHeadDim;
    for (int e = tid; e < TK * (kHeadDim / 8); e += kThreads) {
        const int t = e / (kHeadDim / 8), k8 = e % (kHeadDim / 8);
        float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (t < rows) load8(xbase + static_cast<int64_t>(t) * kHeadDim + k8 * 8, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) xs[(k8 * 8 + j) * TK + t] = v[j];
    }
    __syncthreads();

    // ---- phase 1: hidden activations
    const float* act = xs;   // what phase 2 contracts over
    int act_dim = kHeadDim;
    const WT* wout = static_cast<const WT*>(a.w1) + static_cast<int64_t>(whead) * a.L * kHeadDim;  // linear hash: R
    if (a.hidden > 0) {
        const WT* w1 = static_cast<const WT*>(a.w1) + static_cast<int64_t>(whead) * a.hidden * kHeadDim;
        const WT* b1 = static_cast<const WT*>(a.b1) + static_cast<int64_t>(whead) * a.hidden;
        for (int i = tid; i < a.hidden; i += kThreads) {
            float acc[TK];
            const float bias = load1(b1 + i);
#pragma unroll
            for (int t = 0; t < TK; ++t) acc[t] = bias;
            dot_rows<WT, TK, PF>(w1 + static_cast<int64_t>(i) * kHeadDim, kHeadDim / 8, xs, TK, acc);
#pragma unroll
            for (int t = 0; t < TK; ++t) hs[i * TK + t] = silu(acc[t]);
        }
        __syncthreads();
        act = hs;
        act_dim = a.hidden;
        wout = static_cast<const WT*>(a.w2) + static_cast<int64_t>(whead) * a.L * a.hidden;
    }

    // ---- phase 2: outputs, sign, ballot-pack
    const int lane = tid & 63, wave = tid >> 6;
    const int npairs = (a.W + 1) / 2;
    uint32_t* cbase = a.codes + xhead * a.code_head_stride + (a.code_row0 + r0) * a.W;
    for (int item = wave; item < npairs * KSPLIT; item += kThreads / 64) {
        const int pair = item / KSPLIT, ks = item % KSPLIT;
        const int word = 2 * pair + (lane >> 5);
        const bool live = word < a.W;
        const int o = live ? (31 - (lane & 31)) * a.W + word : 0;
        const WT* row = wout + static_cast<int64_t>(o) * act_dim;
        float y[TK2];
#pragma unroll
        for (int t = 0; t < TK2; ++t) y[t] = 0.0f;
        dot_rows<WT, TK2, PF>(row, act_dim / 8, act + ks * TK2, TK, y);
#pragma unroll
        for (int t = 0; t < TK2; ++t) {
            const unsigned long long m = __ballot(live && (y[t] > 0.0f));
            const int r = ks * TK2 + t;
            if (lane == 0 && r < rows) {
                cbase[static_cast<int64_t>(r) * a.W + 2 * pair] = static_cast<uint32_t>(m);
                if (2 * pair + 1 < a.W) cbase[static_cast<int64_t>(r) * a.W + 2 * pair + 1] = static_cast<uint32_t>(m >> 32);
            }
        }
    }
}

// One vector per workgroup (the query of a head, or the key appended by a decode step), for hidden
// widths that are multiples of 128 (or the linear hash).  Latency matters here, not throughput; the
// work is hashdev::hash_one_vector (hash_vec.h).
// Two independent jobs in one launch (the decode step hashes the queries and the appended keys
// together): workgroups [0, n_first) run job[0], the rest job[1].
struct HashVecArgs {
    HashArgs job[2];
    int n_first;
};

template <typename XT, typename WT, bool PACKED, int T>
__global__ __launch_bounds__(T) void hash_vec_kernel(HashVecArgs jobs)
{
    extern __shared__ __align__(16) float act[];  // hidden activations, or x itself for the linear hash
    const bool second = static_cast<int>(blockIdx.x) >= jobs.n_first;   // uniform over the workgroup
    const HashArgs& a = jobs.job[second ? 1 : 0];
    const int xhead = static_cast<int>(blockIdx.x) - (second ? jobs.n_first : 0);
    hash_one_vector<XT, WT, PACKED, T>(a, xhead, true, threadIdx.x, act, nullptr);
}

// One thread per group of 8 weights of the packed copies (layout: see hash_vec_kernel).
template <typename WT>
__global__ __launch_bounds__(kThreads) void pack_weights_kernel(const WT* __restrict__ w1, const WT* __restrict__ wout,
                                                               WT* __restrict__ pack_w1, WT* __restrict__ pack_out,
                                                               int n_wheads, int hidden, int L)
{
    constexpr int G16 = kHeadDim / 8;
    const int W = L / 32, npairs = (W + 1) / 2;
    const int act_dim = hidden > 0 ? hidden : kHeadDim, n16 = act_dim / kHeadDim;
    const int nib = (hidden + kPackRows - 1) / kPackRows;   // 0 for the linear hash: no first layer
    const int64_t groups1 = static_cast<int64_t>(n_wheads) * nib * G16 * kPackRows;
    const int64_t groups2 = static_cast<int64_t>(n_wheads) * npairs * n16 * G16 * 64;
    const int64_t x = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    const WT* src = nullptr;
    WT* dst;
    if (x < groups1) {
        const int t = static_cast<int>(x % kPackRows), g = static_cast<int>((x / kPackRows) % G16);
        const int ib = static_cast<int>((x / (kPackRows * G16)) % nib), whead = static_cast<int>(x / (static_cast<int64_t>(kPackRows) * G16 * nib));
        const int row = ib * kPackRows + t;
        if (row < hidden) src = w1 + (static_cast<int64_t>(whead) * hidden + row) * kHeadDim + g * 8;
        dst = pack_w1 + x * 8;
    } else if (x < groups1 + groups2) {
        const int64_t y = x - groups1;
        const int lane = static_cast<int>(y % 64), g = static_cast<int>((y / 64) % G16);
        const int r = static_cast<int>((y / (64 * G16)) % n16), pair = static_cast<int>((y / (static_cast<int64_t>(64) * G16 * n16)) % npairs);
        const int whead = static_cast<int>(y / (static_cast<int64_t>(64) * G16 * n16 * npairs));
        const int word = 2 * pair + (lane >> 5);
        if (word < W) {
            const int o = (31 - (lane & 31)) * W + word;
            src = wout + (static_cast<int64_t>(whead) * L + o) * act_dim + r * kHeadDim + g * 8;
        }
        dst = pack_out + y * 8;
    } else {
        return;
    }
    if constexpr (sizeof(WT) == 2) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (src) v = *reinterpret_cast<const uint4*>(src);
        *reinterpret_cast<uint4*>(dst) = v;
    } else {
        float4 v0 = make_float4(0.f, 0.f, 0.f, 0.f), v1 = v0;
        if (src) { v0 = reinterpret_cast<const float4*>(src)[0]; v1 = reinterpret_cast<const float4*>(src)[1]; }
        reinterpret_cast<float4*>(dst)[0] = v0;
        reinterpret_cast<float4*>(dst)[1] = v1;
    }
}

template <typename XT, typename WT>
int run_vec(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, const HashArgs* b, int n_xheads_b, int stage)
{
    const size_t lds = sizeof(float) * (a.hidden > 0 ? a.hidden : kHeadDim);
    HashVecArgs jobs;
    jobs.job[0] = a;
    jobs.job[1] = b ? *b : a;
    jobs.n_first = n_xheads;
    const int grid = n_xheads + (b ? n_xheads_b : 0);
    const bool packed = a.pack_out && (a.hidden == 0 || a.pack_w1) && (!b || (b->pack_out == a.pack_out && b->pack_w1 == a.pack_w1));
    auto kern = packed ? hash_vec_kernel<XT, WT, true, kThreads> : hash_vec_kernel<XT, WT, false, kThreads>;
    int threads = kThreads;
    if constexpr (sizeof(WT) == 2) {
        // Hidden layers of more than 512 units take 256 threads three rounds and more, and their code words
        // two: with a compute unit for every vector, 512 threads shorten both.  128 -> 1024 -> 512: 40
        // vectors 29.7 -> 18.8 us, 160 29.6 -> 19.4 us, 640 44.9 -> 52.2 us (weights from L2 bind it then).
        // No gain at 512 units (11.8 against 11.6 us) or from the arrays as stored (41.7 against 42.4 us),
        // and binary32 rows spill (39.9 against 52.2 us).
        if (packed && a.hidden > 512 && grid <= ctx->n_cus) {
            threads = 512;
            kern = hash_vec_kernel<XT, WT, true, 512>;
        }
    }
    StageTimer timer(ctx, stage);
    timer.launch(kern, dim3(static_cast<unsigned>(grid)), dim3(static_cast<unsigned>(threads)), lds, jobs);
    return hip_rc(hipGetLastError());
}

inline size_t lds_bytes(int tk, int hidden) { return sizeof(float) * tk * (kHeadDim + hidden); }

template <typename XT, typename WT, int TK, int KSPLIT>
int run(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage)
{
    const size_t lds = lds_bytes(TK, a.hidden);
    if (lds > static_cast<size_t>(ctx->max_lds)) return SPOTLIGHT_ERR_UNSUPPORTED;
    auto kern = hash_kernel<XT, WT, TK, KSPLIT>;
    if (allow_dynamic_lds(ctx, reinterpret_cast<const void*>(kern), lds) != SPOTLIGHT_OK) return SPOTLIGHT_ERR_HIP;
    const int64_t tiles = (a.n_rows + TK - 1) / TK;
    dim3 grid(static_cast<unsigned>(tiles), static_cast<unsigned>(n_xheads));
    StageTimer timer(ctx, stage);
    timer.launch(kern, grid, dim3(kThreads), lds, a);
    return hip_rc(hipGetLastError());
}

template <typename XT, typename WT, int TK>
int run_ks(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage)
{
    const int npairs = (a.W + 1) / 2;
    if constexpr (TK >= 4) {
        if (npairs == 1) return run<XT, WT, TK, 4>(ctx, a, n_xheads, stage);
    }
    if constexpr (TK >= 2) {
        if (npairs <= 2) return run<XT, WT, TK, 2>(ctx, a, n_xheads, stage);
    }
    return run<XT, WT, TK, 1>(ctx, a, n_xheads, stage);
}

template <typename XT, typename WT>
int run_tk(spotlight_ctx* ctx, const HashArgs& a, int n_xheads, int stage)
{
    const size_t cap = static_cast<size_t>(ctx->max_lds);
    if constexpr (sizeof(XT) == 2 && sizeof(WT) == 2) {
        if (screened_hash_applies(ctx, a, n_xheads)) return run_screened_hash(ctx, a, n_xheads, stage);
    }
    if (bulk_hash_applies(ctx, a, n_xheads, sizeof(XT), sizeof(WT))) {
        HashArgs all = a;
        all.open = nullptr;   // no first pass has written it
        return run_bulk_hash<XT, WT>(ctx, all, n_xheads, stage);
    }
    // a single vector per head, hidden width a multiple of 128: the latency-oriented kernel
    if (a.n_rows == 1 && a.hidden % kHeadDim == 0) return run_vec<XT, WT>(ctx, a, n_xheads, nullptr, 0, stage);
    if (a.n_rows >= 32 && lds_bytes(32, a.hidden) <= cap) return run_ks<XT, WT, 32>(ctx, a, n_xheads, stage);
    if (a.n_rows >= 4 && lds_bytes(8, a.hidden) <= cap) return run_ks<XT, WT, 8>(ctx, a, n_xheads, stage);
    return run_ks<XT, WT, 1>(ctx, a, n_xheads, stage);
}

}  // namespace

HashArgs make_hash_args(const HashLaunch& h)
{
    HashArgs a;
    a.x = h.x;
    a.x_head_stride = h.x_head_stride;
    a.x_row0 = h.x_row0;
    a.n_rows = h.n_rows;
    a.heads_per_batch = h.heads_per_batch;
    a.group = h.group;
    a.n_wheads = h.heads_per_batch / h.group;
    a.w1 = h.w1;
    a.b1 = h.b1;
    a.w2 = h.w2;
    a.hidden = h.hidden;
    a.L = h.L;
    a.W = h.L / 32;
    a.codes = h.codes;
    a.code_head_stride = h.code_head_stride;
    a.code_row0 = h.code_row0;
    a.zero = h.zero;
    a.zero_words = h.zero_words;
    a.wnorm = h.wnorm;
    a.audit = h.audit;
    a.pack_w1 = h.pack_w1;
    a.pack_out = h.pack_out;
    a.scales = h.scales;
    a.operands = h.operands;
    a.open = h.open;
    a.open_stride = h.open_stride;
    a.open_counts = h.open_counts;
    return a;
}

void pack_sizes(int hidden, int L, size_t* w1_elems, size_t* out_elems)
{
    *w1_elems = *out_elems = 0;
    if (hidden % kHeadDim != 0) return;   // the single-vector kernel takes hidden widths that are multiples of 128 (or 0)
    const int W = L / 32, npairs = (W + 1) / 2;
    const int act_dim = hidden > 0 ? hidden : kHeadDim;
    *w1_elems = static_cast<size_t>((hidden + kPackRows - 1) / kPackRows) * kPackRows * kHeadDim;
    *out_elems = static_cast<size_t>(npairs) * 64 * act_dim;
}

int launch_pack_weights(spotlight_ctx* ctx, const void* w1, const void* w2, int w_dtype, void* pack_w1, void* pack_out)
{
    const Plan& p = ctx->plan;
    const int64_t groups = static_cast<int64_t>(p.Hkv) * (p.pack_w1_elems + p.pack_out_elems) / 8;
    if (groups <= 0) return SPOTLIGHT_OK;
    const void* wout = p.hidden > 0 ? w2 : w1;
    const dim3 grid(static_cast<unsigned>((groups + kThreads - 1) / kThreads));
    if (w_dtype == SPOTLIGHT_BF16)
        hipLaunchKernelGGL(pack_weights_kernel<bf16_raw>, grid, dim3(kThreads), 0, ctx->stream, static_cast<const bf16_raw*>(w1),
                           static_cast<const bf16_raw*>(wout), static_cast<bf16_raw*>(pack_w1), static_cast<bf16_raw*>(pack_out),
                           p.Hkv, p.hidden, p.L);
    else
        hipLaunchKernelGGL(pack_weights_kernel<float>, grid, dim3(kThreads), 0, ctx->stream, static_cast<const float*>(w1),
                           static_cast<const float*>(wout), static_cast<float*>(pack_w1), static_cast<float*>(pack_out), p.Hkv,
                           p.hidden, p.L);
    return hip_rc(hipGetLastError());
}

int launch_hash(spotlight_ctx* ctx, const HashLaunch& h, int stage)
{
    if (h.n_rows <= 0 || h.n_xheads <= 0) return SPOTLIGHT_OK;
    // the weight rows are read 8 elements at a time
    if (h.hidden % 8 != 0) return SPOTLIGHT_ERR_UNSUPPORTED;
    const HashArgs a = make_hash_args(h);
    const bool xb = h.x_dtype == SPOTLIGHT_BF16, wb = h.w_dtype == SPOTLIGHT_BF16;
    if (xb && wb) return run_tk<bf16_raw, bf16_raw>(ctx, a, h.n_xheads, stage);
    if (xb && !wb) return run_tk<bf16_raw, float>(ctx, a, h.n_xheads, stage);
    if (!xb && wb) return run_tk<float, bf16_raw>(ctx, a, h.n_xheads, stage);
    return run_tk<float, float>(ctx, a, h.n_xheads, stage);
}

int launch_hash_pair(spotlight_ctx* ctx, const HashLaunch& h0, const HashLaunch& h1, int stage)
{
    const bool one_launch = h0.n_rows == 1 && h1.n_rows == 1 && h0.n_xheads > 0 && h1.n_xheads > 0 &&
                            h0.hidden == h1.hidden && h0.hidden % kHeadDim == 0 && h0.L == h1.L &&
                            h0.x_dtype == h1.x_dtype && h0.w_dtype == h1.w_dtype;
    if (!one_launch) {
        const int rc = launch_hash(ctx, h0, stage);
        return rc != SPOTLIGHT_OK ? rc : launch_hash(ctx, h1, stage);
    }
    const HashArgs a = make_hash_args(h0), b = make_hash_args(h1);
    const bool xb = h0.x_dtype == SPOTLIGHT_BF16, wb = h0.w_dtype == SPOTLIGHT_BF16;
    if (xb && wb) return run_vec<bf16_raw, bf16_raw>(ctx, a, h0.n_xheads, &b, h1.n_xheads, stage);
    if (xb && !wb) return run_vec<bf16_raw, float>(ctx, a, h0.n_xheads, &b, h1.n_xheads, stage);
    if (!xb && wb) return run_vec<float, bf16_raw>(ctx, a, h0.n_xheads, &b, h1.n_xheads, stage);
    return run_vec<float, float>(ctx, a, h0.n_xheads, &b, h1.n_xheads, stage);
}

}  // namespace spotlight
