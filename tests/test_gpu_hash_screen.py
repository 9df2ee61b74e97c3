"""Bulk hashing in two passes (csrc/hash_screen.h): the first settles most keys on the bfloat16 matrix instructions, the
second hashes the others with the chain.

Codes of whole calls equal the vector-ALU kernel's and, at the rows checked there, the oracle's, at the edges of tiles, rounds
and workgroups, for every kernel of either pass and for values that settle nothing.  What the first pass's bound takes for granted is
checked on its own: how the instructions round, and the norms of the weights against 64 bits."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DEV = "cuda:0"
U = 2.0 ** -24


def _weights(g, H, bits, hidden):
    return [(0.05 * torch.randn(H, *s, generator=g)).bfloat16() for s in ((hidden, 128), (hidden,), (bits, hidden))]


def _check(K, ws, t0, rows, bits, hidden, n_oracle=40, b1_at=0, audit=False):
    """Codes of rows [t0, t0 + rows) both ways; rows outside stay as they were."""
    import paper_2508_19740_amd as sp
    B, H, cap = K.shape[:3]
    Kd, wd = K.to(DEV), [t.to(DEV) for t in ws]
    if b1_at:
        flat = torch.zeros(b1_at + ws[1].numel(), dtype=torch.bfloat16, device=DEV)
        wd[1] = flat[b1_at:].view(ws[1].shape).copy_(wd[1])
    ctx = sp.Spotlight(B, H, H, bits, hidden, cap, 1, kv_dtype=torch.bfloat16, weight_dtype=torch.bfloat16, device=DEV)
    try:
        got = torch.full((B, H, cap, bits // 32), 77, dtype=torch.int32, device=DEV)
        want = got.clone()
        ctx.hash_keys(Kd, *wd, t0, rows, got)
        if audit:
            ctx.set_option(sp.OPT_BULK_HASH_AUDIT, 1)
            again = torch.full_like(got, 5)
            ctx.hash_keys(Kd, *wd, t0, rows, again)
            au = ctx.bulk_hash_audit_read()
            assert torch.equal(again[:, :, t0:t0 + rows], got[:, :, t0:t0 + rows])
            assert au["outputs"] == B * H * rows * bits and au["wrong"] == 0
            ctx.set_option(sp.OPT_BULK_HASH_AUDIT, 0)
        ctx.set_option(sp.OPT_BULK_HASH_MATRIX_CORES, 0)
        ctx.hash_keys(Kd, *wd, t0, rows, want)
        assert torch.equal(got, want)
    finally:
        ctx.close()
    ref = torch.full((B, H, cap, bits // 32), 77, dtype=torch.int32)
    n = min(rows, n_oracle)
    oracle.hash_keys(K, *ws, bits, t0, n, ref)
    assert torch.equal(got[:, :, : t0 + n].cpu(), ref[:, :, : t0 + n])


@pytest.mark.parametrize("bits,hidden", [(32, 16), (64, 32), (96, 48), (128, 128), (160, 112), (256, 128), (64, 144), (128, 256), (192, 256),
                                         (160, 272), (160, 288), (256, 400), (128, 512), (256, 512), (224, 528), (256, 1008), (32, 1024)])
def test_every_instantiation(bits, hidden):
    """Weights of both layers in LDS or a block at a time, one to eight words, every kernel of the second pass."""
    g = torch.Generator().manual_seed(bits + hidden)
    rows = 16400
    _check(torch.randn(1, 8, rows + 6, 128, generator=g).bfloat16(), _weights(g, 8, bits, hidden), 3, rows, bits, hidden)


@pytest.mark.parametrize("B,H,rows", [(1, 1, 131073), (1, 3, 43700), (1, 512, 256), (4, 128, 257), (2, 150, 511), (5, 60, 513), (1, 28, 4703)])
def test_shapes_of_the_grid(B, H, rows):
    """Rounds and ranges that end inside a tile, a round and a span of open rows; more heads than compute units."""
    g = torch.Generator().manual_seed(rows)
    _check(torch.randn(B, H, rows + 2, 128, generator=g).bfloat16(), _weights(g, H, 64, 64), 1, rows, 64, 64, n_oracle=8)


def test_audit_counts_the_first_pass():
    g = torch.Generator().manual_seed(9)
    for bits, hidden in ((128, 256), (256, 512)):
        _check(torch.randn(1, 8, 16384, 128, generator=g).bfloat16(), _weights(g, 8, bits, hidden), 0, 16384, bits, hidden, audit=True)


@pytest.mark.parametrize("bits,hidden", [(128, 256), (256, 512), (96, 80)])
def test_extreme_values(bits, hidden):
    """Padding, keys and rows of weights whose squares underflow or overflow, no numbers, b1 at any element, output rows of
    zeros, all with the codes of the chain; b1 = 0 in one head, where padding has no hidden activation at all."""
    g = torch.Generator().manual_seed(bits)
    H, rows = 8, 16400
    K = torch.randn(1, H, rows, 128, generator=g)
    K[:, :, 100:300] = 0
    K[:, :, 200:230] = -0.0
    K[:, :, 300:340] = torch.ldexp(torch.randn(K[:, :, 300:340].shape, generator=g), torch.tensor(-100))
    K[:, :, 340:380] = torch.ldexp(torch.randn(K[:, :, 340:380].shape, generator=g), torch.tensor(-130))
    K[:, :, 400:440] = torch.ldexp(torch.randn(K[:, :, 400:440].shape, generator=g), torch.tensor(60))
    K[:, :, 440:470] = torch.ldexp(torch.randn(K[:, :, 440:470].shape, generator=g), torch.tensor(120))
    K[:, :, 500:600] = torch.ldexp(K[:, :, 500:600], torch.randint(-40, 40, (1, H, 100, 128), generator=g))
    K[:, :, 5, 3], K[:, :, 6, 9], K[:, :, 7, 1] = float("nan"), float("inf"), -float("inf")
    ws = [t.float() for t in _weights(g, H, bits, hidden)]
    ws[1][1] = 0
    ws[1][2] = -0.0
    ws[2][:, 5:20] = 0
    ws[2][2, 30:40] = torch.ldexp(ws[2][2, 30:40], torch.tensor(-100))
    ws[0][3, 7] = 0
    ws[0][3, 8:12] = torch.ldexp(ws[0][3, 8:12], torch.tensor(-90))
    ws[0][4, 9] = torch.ldexp(ws[0][4, 9], torch.tensor(100))
    ws[2][5, 1, 3] = float("inf")
    ws[1][6, 2] = float("nan")
    ws[1][7] = torch.ldexp(ws[1][7], torch.tensor(20))
    _check(K.bfloat16(), [t.bfloat16().contiguous() for t in ws], 0, rows, bits, hidden, n_oracle=610, b1_at=1)


@pytest.mark.parametrize("bits,hidden", [(64, 64), (256, 512)])
@pytest.mark.parametrize("share", [0.0, 0.5, 1.0])
def test_rows_that_are_all_open(share, bits, hidden):
    """Two equal and opposite halves of a hidden layer make every output a sum that cancels: nothing is settled, and the lists of a
    tile's chains are full.  Scattered among settled rows, or all of them; many workgroups share them (a list holds 512 or 1024 rows)."""
    _check_open_rows(2, 65600, share, bits, hidden)


@pytest.mark.parametrize("bits,hidden", [(64, 64), (96, 256), (160, 64), (256, 128), (256, 512), (32, 1024)])
@pytest.mark.parametrize("share", [0.5, 0.999])
def test_lists_of_open_rows_that_are_full(share, bits, hidden):
    """A workgroup for every head (whole generations of them) has more rows than a list of 2048 holds: it is filled three times, with
    part of a tile in front the second and third time.  Every kernel of the second pass."""
    _check_open_rows(1024, 4133, share, bits, hidden)


def _check_open_rows(H, rows, share, bits, hidden):
    g = torch.Generator().manual_seed(3)
    n, some = hidden // 2, min(H, 8)
    ws = [t.float() for t in _weights(g, some, bits, hidden)]
    ws[0][:, n:], ws[1][:, n:], ws[2][:, :, n:] = ws[0][:, :n], ws[1][:, :n], -ws[2][:, :, :n]
    ws[0][:, ::n], ws[1][:, ::n] = 0, 0
    ws[0][:, 0, 0] = 3.0                                 # the unit that tells the rows apart: a = 3 x_0
    K = torch.randn(1, some, rows, 128, generator=g)
    K[..., 0] = torch.where(torch.rand(1, some, rows, generator=g) < share, torch.tensor(0.0), torch.tensor(4.0))
    again = lambda t, dim: t.bfloat16().repeat_interleave(H // some, dim).contiguous()
    _check(again(K, 1), [again(t, 0) for t in ws], 0, rows, bits, hidden, n_oracle=40 if H == some else 2)


@pytest.mark.parametrize("bits,hidden", [(64, 64), (96, 256), (256, 128), (160, 288), (256, 512), (256, 1008)])
def test_output_rows_of_unequal_norm(bits, hidden):
    """Bounds of each output's own where a word's rows differ: by any factor, by 1e4 once a word, by rows of zeros and of next to
    nothing; equal rows in one head, one word uneven in another."""
    g = torch.Generator().manual_seed(bits + hidden)
    H, rows, W = 8, 16400, bits // 32
    ws = [t.float() for t in _weights(g, H, bits, hidden)]
    ws[2][1] *= torch.exp(1.5 * torch.randn(bits, 1, generator=g))
    ws[2][2, 4 * W:5 * W] *= 1e4
    ws[2][3, 7 * W:30 * W] = 0
    ws[2][4, ::3] = torch.ldexp(ws[2][4, ::3], torch.tensor(-60))
    ws[2][5, W + W // 2] *= 30
    ws[2][6, 2 * W, 5], ws[2][6, 3 * W, 6] = float("inf"), float("nan")
    _check(torch.randn(1, H, rows, 128, generator=g).bfloat16(), [t.bfloat16().contiguous() for t in ws], 0, rows, bits, hidden)


@pytest.mark.parametrize("bits,hidden", [(64, 64), (256, 64), (256, 512)])
@pytest.mark.parametrize("B,H,rows", [(1, 9, 66000), (2, 33, 2100), (1, 200, 700), (1, 1, 70000)])
def test_heads_with_more_open_rows_than_others(B, H, rows, bits, hidden):
    """Every third head has an output that cancels for all keys, another third of them rows that nothing leaves open: the workgroups are
    shared out over the heads by what is open (one workgroup a head where there are many)."""
    g = torch.Generator().manual_seed(H)
    ws, n = [t.float() for t in _weights(g, H, bits, hidden)], hidden // 2
    ws[0][::3, n:], ws[1][::3, n:], ws[2][::3, 5, n:] = ws[0][::3, :n], ws[1][::3, :n], -ws[2][::3, 5, :n]
    K = torch.randn(B, H, rows, 128, generator=g)
    ws[1][1::3] = 0
    K[:, 1::3] = 0
    _check(K.bfloat16(), [t.bfloat16().contiguous() for t in ws], 0, rows, bits, hidden, n_oracle=8)


@pytest.mark.parametrize("n_open", [1, 2, 3, 15, 16, 17])
def test_lists_of_every_length(n_open):
    """The same of a few output rows, 288 to 512 hidden units and long codes: 32 to 544 outputs of a tile on its list of 512, run by one
    wavefront or by all, the last with no room for some."""
    g = torch.Generator().manual_seed(n_open)
    bits, hidden, H, rows = 256, 512, 2, 33000
    n = hidden // 2
    ws = [t.float() for t in _weights(g, H, bits, hidden)]
    ws[0][:, n:], ws[1][:, n:], ws[2][:, 7:7 + n_open, n:] = ws[0][:, :n], ws[1][:, :n], -ws[2][:, 7:7 + n_open, :n]
    _check(torch.randn(1, H, rows, 128, generator=g).bfloat16(), [t.bfloat16().contiguous() for t in ws], 0, rows, bits, hidden)


def test_profile_counts_a_call_once():
    import paper_2508_19740_amd as sp
    g = torch.Generator().manual_seed(1)
    K, ws = torch.randn(1, 8, 16384, 128, generator=g).bfloat16().to(DEV), [t.to(DEV) for t in _weights(g, 8, 128, 256)]
    codes = torch.zeros(1, 8, 16384, 4, dtype=torch.int32, device=DEV)
    ctx = sp.Spotlight(1, 8, 8, 128, 256, 16384, 1, kv_dtype=torch.bfloat16, weight_dtype=torch.bfloat16, device=DEV)
    try:
        ctx.profile_enable(True)
        ctx.hash_keys(K, *ws, 0, 16384, codes)
        ms, n = ctx.profile_read()["hash_keys"]
        assert n == 1 and ms > 0
    finally:
        ctx.close()


def test_profile_times_every_launch_of_a_call():
    """512 weight heads that are used for 256 keys each: what a call does with the weights first is a good part of it.  The times of its
    launches sum to the call's but for the gaps between them."""
    import paper_2508_19740_amd as sp
    g = torch.Generator().manual_seed(1)
    H, rows, bits, hidden = 512, 256, 32, 1024
    K, ws = torch.randn(1, H, rows, 128, generator=g).bfloat16().to(DEV), [t.to(DEV) for t in _weights(g, H, bits, hidden)]
    codes = torch.zeros(1, H, rows, 1, dtype=torch.int32, device=DEV)
    ctx = sp.Spotlight(1, H, H, bits, hidden, rows, 1, kv_dtype=torch.bfloat16, weight_dtype=torch.bfloat16, device=DEV)
    try:
        def whole():
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(10):
                ctx.hash_keys(K, *ws, 0, rows, codes)
            stop.record()
            torch.cuda.synchronize()
            return start.elapsed_time(stop) / 10
        whole()
        call = min(whole() for _ in range(3))
        ctx.profile_enable(True)
        for _ in range(10):
            ctx.hash_keys(K, *ws, 0, rows, codes)
        ms, n = ctx.profile_read()["hash_keys"]
        print(f"[profile] call {call * 1e3:.1f} us, its launches {ms / n * 1e3:.1f}")
        assert n == 10 and ms / n > 0.9 * call
    finally:
        ctx.close()


@pytest.mark.parametrize("bits,hidden", [(128, 256), (256, 512), (512, 0)])
def test_in_a_hip_graph(bits, hidden):
    """Both passes (and the linear hash) recorded once and replayed over other keys, with eager work between the replays."""
    import paper_2508_19740_amd as sp
    g = torch.Generator().manual_seed(bits)
    ws = _weights(g, 8, bits, hidden) if hidden else [(0.1 * torch.randn(8, bits, 128, generator=g)).bfloat16()]
    ws = [t.to(DEV) for t in ws] + ([] if hidden else [None, None])
    keys = [torch.randn(1, 8, 16400, 128, generator=g).bfloat16().to(DEV) for _ in range(3)]
    K = keys[0].clone()
    codes, want = (torch.zeros(1, 8, 16400, bits // 32, dtype=torch.int32, device=DEV) for _ in range(2))
    ctx = sp.Spotlight(1, 8, 8, bits, hidden, 16400, 1, kv_dtype=torch.bfloat16, weight_dtype=torch.bfloat16, device=DEV)
    try:
        ctx.hash_keys(K, *ws, 0, 16400, codes)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ctx.hash_keys(K, *ws, 0, 16400, codes)
        for k in (keys[1], keys[2], keys[0], keys[1]):
            K.copy_(k)
            codes.zero_()
            graph.replay()
            torch.cuda.synchronize()
            ctx.hash_keys(k, *ws, 0, 16400, want)
            torch.cuda.synchronize()
            assert torch.equal(codes, want)
    finally:
        ctx.close()


# ------------------------------------------------------------------ what the bound takes for granted
PROBE = r"""
#include "hash_screen.h"
using namespace spotlight;
__global__ void product(const uint16_t* A, const uint16_t* B, const float* C, float* D)
{
    const int64_t i = blockIdx.x;
    const int l = threadIdx.x, c = l & 31, h = l >> 5;
    const bulk::bf16x8_t a = *reinterpret_cast<const bulk::bf16x8_t*>(A + (i * 32 + c) * 16 + 8 * h), b = *reinterpret_cast<const bulk::bf16x8_t*>(B + (i * 32 + c) * 16 + 8 * h);
    bulk::f32x16_t acc;
    for (int v = 0; v < 16; ++v) acc[v] = C[(i * 32 + 8 * (v / 4) + 4 * h + v % 4) * 32 + c];
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
    for (int v = 0; v < 16; ++v) D[(i * 32 + 8 * (v / 4) + 4 * h + v % 4) * 32 + c] = acc[v];
}
__global__ void activation(const float* a, float* chain, float* fast, float* hi, float* lo, int n)
{
    const int i = (blockIdx.x * 64 + threadIdx.x) * 8;
    if (i >= n) return;
    float h[8];
    for (int e = 0; e < 8; ++e) { chain[i + e] = hashdev::silu(a[i + e]); fast[i + e] = h[e] = screen::fast_silu(a[i + e]); }
    bulk::bf16x8_t p, q;
    screen::split8(h, p, q);
    for (int e = 0; e < 8; ++e) { hi[i + e] = static_cast<float>(p[e]); lo[i + e] = static_cast<float>(q[e]); }
}
extern "C" int run_product(const void* A, const void* B, const void* C, void* D, int n)
{
    product<<<n, 64>>>((const uint16_t*)A, (const uint16_t*)B, (const float*)C, (float*)D);
    return hipDeviceSynchronize();
}
extern "C" int run_activation(const void* a, void* chain, void* fast, void* hi, void* lo, int n)
{
    activation<<<n / 512, 64>>>((const float*)a, (float*)chain, (float*)fast, (float*)hi, (float*)lo, n);
    return hipDeviceSynchronize();
}
extern "C" int run_scales(const void* w1, const void* b1, const void* w2, void* out, int heads, int hidden, int L)
{
    using hashdev::bf16_raw;
    screen::scales_kernel<8><<<dim3(heads, 1 + L / 32), kThreads>>>((const bf16_raw*)w1, (const bf16_raw*)b1, (const bf16_raw*)w2, (char*)out, nullptr, nullptr, 0, hidden, L);
    return hipDeviceSynchronize();
}
"""


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    from paper_2508_19740_amd import build
    tmp = tmp_path_factory.mktemp("probe")
    src, lib = tmp / "probe.hip", tmp / "probe.so"
    src.write_text(PROBE)
    subprocess.run(["/opt/rocm/bin/hipcc", *build.FLAGS, "-shared", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC, "-o", str(lib), str(src)],
                   check=True, capture_output=True)
    return ctypes.CDLL(str(lib))


def _p(t):
    return ctypes.c_void_p(t.data_ptr())


@pytest.mark.parametrize("spread", [0, 3, 8, 20])
@pytest.mark.parametrize("low_bits", [False, True])
def test_rounding_of_the_matrix_instruction(probe, spread, low_bits):
    """r of a group of eight products and c is within u (10 max|p| + 2 |c| + |r|) of the exact sum (64 bits hold it:
    exponents within 2 * 20 of each other and 16-bit products).  Groups: k = 0 .. 7, then 8 .. 15; one at a time here."""
    g = np.random.default_rng(spread + 100 * low_bits)
    n = 500

    def values(shape, s):
        m = (255 if low_bits else 128 + g.integers(0, 128, shape)) / 128.0
        return torch.tensor(g.choice([-1.0, 1.0], shape) * m * np.exp2(g.integers(-s, s + 1, shape).astype(np.float64)), dtype=torch.float64)

    for first in (0, 8):
        A, B = values((n, 32, 16), spread), values((n, 32, 16), spread)
        A[:, :, 8 - first:16 - first] = 0
        C = values((n, 32, 32), 2 * spread) * torch.tensor(g.random((n, 32, 32)) + 0.5)
        C[: n // 4] = 0
        s = torch.matmul(A, B.transpose(1, 2))
        C[n // 4: n // 2] = -s[n // 4: n // 2] * (1 + 1e-6)     # cancellation
        C = C.float()
        ad, bd, cd = A.bfloat16().to(DEV), B.bfloat16().to(DEV), C.to(DEV)
        D = torch.empty_like(cd)
        assert probe.run_product(_p(ad), _p(bd), _p(cd), _p(D), n) == 0
        D, C = D.cpu().double(), C.double()
        biggest = (A.abs().unsqueeze(2) * B.abs().unsqueeze(1)).amax(-1)
        err, bound = (D - (s + C)).abs(), U * (10 * biggest + 2 * C.abs() + D.abs())
        assert (err <= bound).all(), (err / bound).max()


def _product(probe, A, B, C):
    ad, bd, cd = A.bfloat16().to(DEV), B.bfloat16().to(DEV), C.float().to(DEV)
    D = torch.empty_like(cd)
    assert probe.run_product(_p(ad), _p(bd), _p(cd), _p(D), len(A)) == 0
    return D.cpu().double()


@pytest.mark.parametrize("apart", [-20, -8, -1, 0, 1, 8, 20])
@pytest.mark.parametrize("spread", [0, 3, 8])
def test_rounding_with_both_groups_filled(probe, spread, apart):
    """The second group adds to the first's rounded sum: r1 of c + products 0 .. 7, r of r1 + products 8 .. 15, each within
    u (10 max|p| + 2 |addend| + |result|).  Magnitudes of the groups apart by 2^apart; c takes the first group's sum away, or both; the
    second group takes the first's away, as it is and but for one product."""
    g = np.random.default_rng(spread + 100 * (apart + 50))
    n = 640

    def values(shape, s):
        m = (128 + g.integers(0, 128, shape)) / 128.0
        return torch.tensor(g.choice([-1.0, 1.0], shape) * m * np.exp2(g.integers(-s, s + 1, shape).astype(np.float64)), dtype=torch.float64)

    A, B = values((n, 32, 16), spread), values((n, 32, 16), spread)
    A[:, :, 8:] *= 2.0 ** apart
    C = values((n, 32, 32), 2 * spread) * torch.tensor(g.random((n, 32, 32)) + 0.5) * torch.tensor(np.exp2(g.choice([0, apart], (n, 32, 32)).astype(np.float64)))
    A[4 * n // 8:, :, 8:] = -A[4 * n // 8:, :, :8]             # the second group takes the first's sum away (with c in between)
    B[4 * n // 8:, :, 8:] = B[4 * n // 8:, :, :8]
    A[6 * n // 8:, :, 15] *= 2.0 ** apart
    products = lambda lo: torch.matmul(A[:, :, lo:lo + 8], B[:, :, lo:lo + 8].transpose(1, 2))
    biggest = lambda lo: (A[:, :, lo:lo + 8].abs().unsqueeze(2) * B[:, :, lo:lo + 8].abs().unsqueeze(1)).amax(-1)
    s1, s2 = products(0), products(8)
    C[: n // 8] = 0
    C[n // 8: 2 * n // 8] = -s1[n // 8: 2 * n // 8] * (1 + 1e-6)
    C[2 * n // 8: 3 * n // 8] = -(s1 + s2)[2 * n // 8: 3 * n // 8] * (1 + 1e-6)
    C[5 * n // 8: 6 * n // 8] = 0
    C[6 * n // 8: 7 * n // 8] = -s1[6 * n // 8: 7 * n // 8]
    C = C.float().double()
    D = _product(probe, A, B, C)
    first = (C + s1).abs()
    err1 = U * (10 * biggest(0) + 2 * C.abs() + 1.001 * first)
    err, bound = (D - (C + s1 + s2)).abs(), 1.001 * (err1 + U * (10 * biggest(8) + 2 * (first + err1) + D.abs()))
    print(f"[error / bound] spread {spread}, apart {apart}: {(err / bound).max():.3f}")
    assert (err <= bound).all(), (err / bound).max()


def test_order_of_the_matrix_instruction(probe):
    """Products 0 .. 7 come first, and their sum with c is rounded before 8 .. 15 come: where one of the first takes c away
    exactly, the others lose nothing to it."""
    g = np.random.default_rng(1)
    n = 8 * 40
    A, B = (torch.tensor(g.choice([-1.0, 1.0], (n, 32, 16)) * (128 + g.integers(0, 128, (n, 32, 16))) / 128.0) for _ in range(2))
    A[:, :, :8] = 0
    for k in range(8):
        A[k::8, :, k], B[k::8, :, k] = 2.0 ** 20, 2.0 ** 10
    C = torch.full((n, 32, 32), -2.0 ** 30, dtype=torch.float64)
    s2 = torch.matmul(A[:, :, 8:], B[:, :, 8:].transpose(1, 2))
    biggest = (A[:, :, 8:].abs().unsqueeze(2) * B[:, :, 8:].abs().unsqueeze(1)).amax(-1)
    D = _product(probe, A, B, C)
    err, bound = (D - s2).abs(), U * (10 * biggest + D.abs())
    assert (err <= bound).all(), (err / bound).max()


def test_activations(probe):
    """Both evaluations of SiLU within 12 u |h| + 2 u |a| of each other; hi + lo within 128 u |h| of the activation."""
    g = torch.Generator().manual_seed(5)
    n = 1 << 20
    a = torch.cat([torch.linspace(-100, 100, n // 2), torch.randn(n // 4, generator=g), torch.exp2(torch.empty(n // 8).uniform_(-90, 90, generator=g)),
                   -torch.exp2(torch.empty(n // 8).uniform_(-90, 90, generator=g))]).to(DEV)
    chain, fast, hi, lo = (torch.empty_like(a) for _ in range(4))
    assert probe.run_activation(_p(a), _p(chain), _p(fast), _p(hi), _p(lo), n) == 0
    a, chain, fast, hi, lo = (t.double() for t in (a, chain, fast, hi, lo))
    assert ((chain - fast).abs() <= U * (12 * fast.abs() + 2 * a.abs()) + 1e-30).all()
    assert ((hi + lo - fast).abs() <= 128 * U * fast.abs() + 1e-37).all()


@pytest.mark.parametrize("heads,bits,hidden", [(3, 32, 16), (2, 96, 48), (2, 128, 256), (1, 256, 1008)])
def test_scales(probe, heads, bits, hidden):
    """The norms of the bound: never below those of the stored weights in 64 bits, and no more than 0.3 % above."""
    g = torch.Generator().manual_seed(bits + hidden)
    ws = _weights(g, heads, bits, hidden)
    ws[2][:, 3] = 0
    ws[1][0] = 0
    W = bits // 32
    flat = torch.zeros(heads * ((1 + W) * 4 + W * 64), dtype=torch.float32, device=DEV)   # records, then two norms of every output
    wd = [t.to(DEV) for t in ws]
    assert probe.run_scales(*(_p(t) for t in wd), _p(flat), heads, hidden, bits) == 0
    out, each = flat[:heads * (1 + W) * 4].view(heads, 1 + W, 4).cpu(), flat[heads * (1 + W) * 4:].view(heads, W, 32, 2).double().cpu()
    w1, b1, w2 = (t.double() for t in ws)
    k = torch.arange(128) % 32     # partial sums charged to a product, and its part in the groups' (recounted here)
    t1 = torch.zeros(128, dtype=torch.float64)
    for s in range(0, 32):         # sums after term s + 1 of a stretch of 32: the first half reaches back, the second forward
        t1 += ((k <= s) if s < 16 else (k > s)).double()
        if s % 8 == 7:
            t1 += 3 * ((k <= s) if s < 16 else (k > s)).double()
    t1 += 10
    i = torch.arange(hidden)
    s2 = torch.zeros(hidden, dtype=torch.float64)
    for s in range(hidden):
        s2 += ((i <= s) if s < hidden // 2 else (i > s)).double()
    s2 = s2 * 1.75 + 151
    want1 = [(t1 * w1).square().sum((1, 2)).sqrt(), (t1 * w1).square().sum(2).sqrt().amax(1), b1.square().sum(1).sqrt()]
    for e in range(3):
        got = out[:, 0, e].double()
        assert (got >= want1[e]).all() and (got <= 1.003 * want1[e] + 1e-11).all(), (e, got, want1[e])
    assert (out[:, 0, 3].view(torch.int32) == torch.tensor([1] + [0] * (heads - 1))).all()
    rows = (torch.arange(32).view(32, 1) * (bits // 32) + torch.arange(bits // 32)).t()     # [word][c]
    want_s = U * (s2 * w2).square().sum(2).sqrt()[:, rows].amax(2)
    want_w = w2.square().sum(2).sqrt()[:, rows].amax(2)
    for e, want in ((0, want_s), (1, want_w)):
        got = out[:, 1:, e].double()
        assert (got >= want).all() and (got <= (1.003 + 2.2 * (e == 0) / hidden) * want + 1e-11).all(), (e, got, want)
    zeros = out[:, 1:, 2].contiguous().view(torch.int32)
    for word in range(bits // 32):
        mask = sum(1 << c for c in range(32) if rows[word, c] == 3)
        assert (zeros[:, word] == mask).all()
    for e, want in ((0, U * (s2 * w2).square().sum(2).sqrt()[:, rows]), (1, w2.square().sum(2).sqrt()[:, rows])):
        assert (each[..., e] >= want).all() and (each[..., e] <= (1.003 + 2.2 * (e == 0) / hidden) * want + 1e-11).all(), e
    assert (out[:, 1:, 3].view(torch.int32) == 0).all()           # rows of much the same norm


def test_rows_of_unequal_norm_are_marked(probe):
    """Uneven: the largest norm more than 1.5 times a row's in the mean, rows of zeros left out."""
    heads, bits, hidden = 6, 64, 48
    g = torch.Generator().manual_seed(4)
    ws = _weights(g, heads, bits, hidden)
    w2 = torch.ones(heads, bits, hidden)
    w2[1, 6] = 1.45                                               # output 6: word 0
    w2[2, 7] = 1.6                                                # output 7: word 1
    w2[3, 2:] = 0
    w2[4, 8] = 1e-20
    w2[5, 9, 0] = float("nan")
    ws[2] = w2.bfloat16()
    flat = torch.zeros(heads * (3 * 4 + 2 * 64), dtype=torch.float32, device=DEV)
    wd = [t.to(DEV) for t in ws]
    assert probe.run_scales(*(_p(t) for t in wd), _p(flat), heads, hidden, bits) == 0
    uneven = flat[:heads * 12].view(heads, 3, 4)[:, 1:, 3].contiguous().view(torch.int32)
    assert uneven.tolist() == [[0, 0], [0, 0], [0, 1], [0, 0], [1, 0], [0, 1]]
