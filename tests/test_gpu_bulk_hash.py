"""The bulk hash on the matrix cores at the edges of its dispatch: every kernel instantiation (hidden
widths around the blocks a wavefront owns, code lengths around the words it owns, the linear hash,
1024-bit codes, both types of keys and weights), row counts around a tile and a run of tiles, and
values that separate a chain of correctly rounded fused multiply-adds from anything else.  The whole
code tensor equals the vector-ALU kernel's (SPOTLIGHT_OPT_BULK_HASH_MATRIX_CORES = 0) and, at the
rows checked there, the oracle's, bit for bit."""
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _both(B, H, rows, t0, cap, bits, hidden, kv, w, stress=False, seed=3, b1_at=0):
    import paper_2508_19740_amd as sp
    g = torch.Generator().manual_seed(seed + rows + bits + hidden)
    K = torch.randn(B, H, cap, 128, generator=g)
    if hidden:
        ws = [0.05 * torch.randn(H, *s, generator=g) for s in ((hidden, 128), (hidden,), (bits, hidden))]
    else:
        ws = [0.05 * torch.randn(H, bits, 128, generator=g)]
    if stress:   # exponents over the whole range in both factors: products that are denormal, sums that cancel or overflow
        K = torch.ldexp(K, torch.randint(-75, 60, K.shape, generator=g))
        ws[0] = torch.ldexp(ws[0], torch.randint(-75, 60, ws[0].shape, generator=g))
        K[:, :, :: 7] = torch.ldexp(torch.randn(K[:, :, ::7].shape, generator=g), torch.tensor(-70))
        K[:, :, 100:140] = torch.ldexp(torch.randn(K[:, :, 100:140].shape, generator=g), torch.tensor(-100))   # squares underflow
        K[:, :, 200:240] = torch.ldexp(torch.randn(K[:, :, 200:240].shape, generator=g), torch.tensor(-130))   # denormal
        K[:, :, 300:340] = 0
        ws[-1][:, 3:9] = torch.ldexp(ws[-1][:, 3:9], torch.tensor(-100))
        K[:, :, 5, 3], K[:, :, 6, 9] = float("nan"), float("inf")
    K = K.to(DT[kv])
    ws = [t.to(DT[w]).contiguous() for t in ws] + ([None, None] if not hidden else [])
    dev = torch.device("cuda:0")
    Kd, wd = K.to(dev), [None if t is None else t.to(dev) for t in ws]
    if b1_at:   # a slice of a larger buffer that starts at this element
        flat = torch.zeros(b1_at + ws[1].numel(), dtype=DT[w], device=dev)
        wd[1] = flat[b1_at:].view(ws[1].shape).copy_(wd[1])
        assert wd[1].data_ptr() % 16 != 0 and wd[1].is_contiguous()
    ctx = sp.Spotlight(B, H, H, bits, hidden, cap, 1, kv_dtype=DT[kv], weight_dtype=DT[w], device=dev)
    try:
        got = torch.full((B, H, cap, bits // 32), 77, dtype=torch.int32, device=dev)
        want = got.clone()
        ctx.hash_keys(Kd, *wd, t0, rows, got)
        ctx.set_option(sp.OPT_BULK_HASH_MATRIX_CORES, 0)
        ctx.hash_keys(Kd, *wd, t0, rows, want)
        assert torch.equal(got, want)
    finally:
        ctx.close()
    n = min(rows, 350 if stress else 70)
    ref = torch.full((B, H, cap, bits // 32), 77, dtype=torch.int32)
    oracle.hash_keys(K, *ws, bits, t0, n, ref)
    assert torch.equal(got[:, :, : t0 + n].cpu(), ref[:, :, : t0 + n])


@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("w", ["bf16", "f32"])
@pytest.mark.parametrize("bits,hidden", [
    (32, 16), (64, 32), (96, 48), (128, 128), (160, 144), (256, 128), (512, 112),     # one block a wavefront
    (128, 256), (128, 176), (256, 256), (480, 256), (64, 200),                        # two
    (256, 512), (128, 264), (512, 384), (160, 520),                                   # eight wavefronts
    (512, 1024), (128, 640), (288, 1040), (64, 1112), (64, 1152),                     # up to what LDS holds, and past it
    (128, 0), (32, 0), (512, 0), (224, 0), (1024, 0), (1024, 256),                    # linear, 1024 bits
])
def test_every_instantiation(bits, hidden, kv, w):
    _both(1, 2, 33, 3, 40, bits, hidden, kv, w)


@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("w", ["bf16", "f32"])
@pytest.mark.parametrize("bits,hidden", [(128, 256), (256, 128), (256, 512), (128, 264), (512, 1024), (64, 1112)])
def test_biases_at_any_element(bits, hidden, kv, w):
    """W1 and W2 are 16-byte aligned, b1 need not be."""
    _both(1, 2, 33, 3, 40, bits, hidden, kv, w, b1_at=1)


@pytest.mark.parametrize("rows", [8, 9, 16, 17, 31, 32, 63, 64, 65, 511, 513, 2049])
@pytest.mark.parametrize("bits,hidden", [(128, 256), (128, 0), (256, 512)])
def test_row_counts(rows, bits, hidden):
    _both(3, 2, rows, 5, rows + 9, bits, hidden, "bf16", "bf16")


def test_runs_of_several_tiles():
    _both(2, 32, 16 * 32 * 6 + 1, 0, 16 * 32 * 6 + 1, 128, 256, "bf16", "bf16")
    _both(2, 32, 16 * 32 * 6 + 1, 0, 16 * 32 * 6 + 1, 96, 0, "f32", "bf16")


@pytest.mark.parametrize("bits,hidden,w", [(96, 64, "f32"), (64, 64, "bf16"), (96, 0, "bf16")])
@pytest.mark.parametrize("rows", [90, 600])
def test_runs_that_do_not_divide(rows, bits, hidden, w):
    """512 heads of 3 and of 19 tiles: runs of one, and of ten and nine."""
    _both(16, 32, rows, 0, rows, bits, hidden, "bf16", w)


@pytest.mark.parametrize("B,rows,bits,hidden,w", [(1, 31, 512, 64, "f32"), (1, 32, 512, 64, "f32"), (10, 24, 32, 264, "bf16"), (10, 25, 32, 264, "bf16"),
                                                  (10, 65, 512, 16, "f32"), (10, 65, 480, 16, "f32"), (10, 65, 1024, 24, "bf16")])
def test_calls_of_either_kernel(B, rows, bits, hidden, w):
    _both(B, 30 if B > 1 else 3, rows, 2, rows + 5, bits, hidden, "bf16", w)


def test_many_heads_of_few_rows():
    """More heads than compute units: the row count from which the matrix cores take over is another."""
    _both(10, 30, 16, 1, 20, 64, 128, "bf16", "bf16")
    _both(10, 30, 17, 1, 20, 64, 128, "bf16", "bf16")


@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("bits,hidden", [(128, 256), (32, 136), (64, 200)])
def test_two_blocks_a_wavefront_with_more_tiles_than_compute_units(bits, hidden, kv):
    _both(10, 30, 33, 1, 36, bits, hidden, kv, "f32")
    _both(10, 30, 33, 1, 36, bits, hidden, kv, "bf16")


@pytest.mark.parametrize("rows", [31, 32])
@pytest.mark.parametrize("bits,hidden", [(64, 256), (32, 160), (64, 512), (96, 256)])
def test_short_codes_of_few_rows(rows, bits, hidden):
    """Up to 64 bits behind a wide hidden layer: few rows stay with the tiles of 8."""
    _both(1, 2, rows, 3, 40, bits, hidden, "bf16", "bf16")
    _both(1, 2, rows, 3, 40, bits, hidden, "f32", "f32")


@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("bits,hidden", [(128, 0), (512, 0), (128, 256), (256, 512)])
def test_audit(bits, hidden, kv):
    """The audited call writes the same codes, counts every output of every row, and finds none settled wrongly."""
    import paper_2508_19740_amd as sp
    g = torch.Generator().manual_seed(bits + hidden)
    dev = torch.device("cuda:0")
    K = torch.randn(1, 2, 1000, 128, generator=g).to(DT[kv]).to(dev)
    ws = [0.05 * torch.randn(2, *s, generator=g) for s in ((((hidden, 128), (hidden,), (bits, hidden))) if hidden else ((bits, 128),))]
    ws = [t.bfloat16().to(dev) for t in ws] + ([None, None] if not hidden else [])
    ctx = sp.Spotlight(1, 2, 2, bits, hidden, 1000, 1, kv_dtype=DT[kv], weight_dtype=torch.bfloat16, device=dev)
    try:
        got = torch.zeros(1, 2, 1000, bits // 32, dtype=torch.int32, device=dev)
        want = got.clone()
        ctx.hash_keys(K, *ws, 0, 999, want)
        ctx.set_option(sp.OPT_BULK_HASH_AUDIT, 1)
        ctx.hash_keys(K, *ws, 0, 999, got)
        au = ctx.bulk_hash_audit_read()
        assert torch.equal(got, want)
        assert au["outputs"] == 2 * 999 * bits and au["wrong"] == 0
        assert 0 < au["listed"] < au["outputs"] // 50 and 0.0 < au["max_ratio"] < au["eps"]
    finally:
        ctx.close()


@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("bits,hidden", [(128, 0), (512, 0), (128, 256), (96, 112), (256, 512), (352, 48), (512, 1024)])
def test_zeros_are_settled(bits, hidden, kv):
    """A vector of zeros (padding; b1 = 0) and an output row of zeros (a code filled up) are settled as they
    stand: none of their outputs is recomputed, alone or together.  A vector whose squares underflow is not
    zeros: all its outputs are."""
    import paper_2508_19740_amd as sp
    g = torch.Generator().manual_seed(bits + hidden)
    dev = torch.device("cuda:0")
    n = 300
    x = torch.randn(1, 2, n, 128, generator=g)
    ws = [0.05 * torch.randn(2, *s, generator=g) for s in (((hidden, 128), (hidden,), (bits, hidden)) if hidden else ((bits, 128),))]
    if hidden:
        ws[1].zero_()
    ws[-1][:, 5:bits:3] = -0.0
    zero = torch.zeros_like(x)
    zero[:, :, ::2] = -0.0
    tiny = torch.zeros_like(x)
    tiny[..., 77] = 1e-30
    live = torch.count_nonzero(ws[-1][0].abs().sum(-1)).item()              # outputs of a head that are not zero rows
    wd = [t.bfloat16().to(dev) for t in ws] + ([None, None] if not hidden else [])
    ctx = sp.Spotlight(1, 2, 2, bits, hidden, n, 1, kv_dtype=DT[kv], weight_dtype=torch.bfloat16, device=dev)
    try:
        ctx.set_option(sp.OPT_BULK_HASH_AUDIT, 1)
        for keys, least, most in ((zero, 0, 0), (x, 0, 2 * n * live // 50), (tiny, 2 * n * bits, 2 * n * bits)):
            got = torch.full((1, 2, n, bits // 32), -1, dtype=torch.int32, device=dev)
            ctx.hash_keys(keys.to(DT[kv]).to(dev), *wd, 0, n, got)
            au = ctx.bulk_hash_audit_read()
            assert au["outputs"] == 2 * n * bits and au["wrong"] == 0 and least <= au["listed"] <= most, au
            want = torch.zeros(1, 2, n, bits // 32, dtype=torch.int32)
            oracle.hash_keys(keys.to(DT[kv]), *[t.bfloat16() for t in ws], *([None, None] if not hidden else []), bits, 0, n, want)
            assert torch.equal(got.cpu(), want)
    finally:
        ctx.close()


@pytest.mark.parametrize("bits,hidden,kv,w", [(128, 256, "f32", "f32"), (64, 128, "bf16", "bf16"), (128, 256, "bf16", "bf16"), (512, 0, "f32", "f32"),
                                              (512, 0, "bf16", "bf16"), (128, 0, "f32", "bf16"), (256, 512, "f32", "bf16")])
def test_extreme_values(bits, hidden, kv, w):
    _both(1, 2, 700, 0, 700, bits, hidden, kv, w, stress=True)


@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("bits,hidden", [(128, 256), (32, 144), (96, 192)])
@pytest.mark.parametrize("B,rows", [(1, 9), (8, 17), (8, 32), (8, 33)])
def test_up_to_a_tile_for_every_compute_unit(B, rows, bits, hidden, kv):
    """Certified words with a block of hidden units for each of eight wavefronts, 256 tiles at most, and the step to four."""
    _both(B, 32, rows, 2, rows + 4, bits, hidden, kv, "bf16")


@pytest.mark.parametrize("kv,w", [("f32", "f32"), ("bf16", "f32"), ("f32", "bf16"), ("bf16", "bf16")])
@pytest.mark.parametrize("B,H,rows", [(1, 4, 10007), (1, 28, 700), (2, 150, 129)])
def test_runs_that_differ_by_a_tile(B, H, rows, kv, w):
    _both(B, H, rows, 0, rows, 128, 256, kv, w)
