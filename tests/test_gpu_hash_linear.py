"""The linear hash of larger calls (hash_linear_tiles_kernel): codes equal the vector-ALU kernel's over the whole call and, at
the rows checked there, the oracle's: word counts around its groups of four and sixteen, ends inside a tile, a
round and a workgroup, values that leave everything open (lists that overflow), zeros, and what the audit counts."""
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DT = {"f32": torch.float32, "bf16": torch.bfloat16}
DEV = "cuda:0"


def _check(K, r, t0, rows, bits, n_oracle=40, audit=False):
    import paper_2508_19740_amd as sp
    B, H, cap = K.shape[:3]
    Kd, rd = K.to(DEV), r.to(DEV)
    ctx = sp.Spotlight(B, H, H, bits, 0, cap, 1, kv_dtype=K.dtype, weight_dtype=torch.bfloat16, device=DEV)
    try:
        got = torch.full((B, H, cap, bits // 32), 77, dtype=torch.int32, device=DEV)
        want, au = got.clone(), None
        ctx.hash_keys(Kd, rd, None, None, t0, rows, got)
        if audit:
            ctx.set_option(sp.OPT_BULK_HASH_AUDIT, 1)
            again = torch.full_like(got, 77)
            ctx.hash_keys(Kd, rd, None, None, t0, rows, again)
            au = ctx.bulk_hash_audit_read()
            ctx.set_option(sp.OPT_BULK_HASH_AUDIT, 0)
            assert torch.equal(again, got)
            assert au["outputs"] == B * H * rows * bits and au["wrong"] == 0 and au["max_ratio"] < au["eps"]
        ctx.set_option(sp.OPT_BULK_HASH_MATRIX_CORES, 0)
        ctx.hash_keys(Kd, rd, None, None, t0, rows, want)
        assert torch.equal(got, want)
    finally:
        ctx.close()
    ref = torch.full((B, H, cap, bits // 32), 77, dtype=torch.int32)
    n = min(rows, n_oracle)
    oracle.hash_keys(K, r, None, None, bits, t0, n, ref)
    assert torch.equal(got[:, :, : t0 + n].cpu(), ref[:, :, : t0 + n])
    return au


def _inputs(B, H, cap, bits, kv, seed=1):
    g = torch.Generator().manual_seed(seed + bits)
    return torch.randn(B, H, cap, 128, generator=g).to(DT[kv]), (0.1 * torch.randn(H, bits, 128, generator=g)).bfloat16()


@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("bits,H,rows", [(32, 2, 32801), (64, 2, 16390), (96, 3, 11000), (128, 2, 16447), (160, 4, 8250), (480, 2, 16400), (512, 2, 4097),
                                         (512, 300, 257), (128, 200, 511), (1024, 2, 31), (1024, 2, 33), (1024, 3, 1030), (512, 40, 513)])
def test_shapes(bits, H, rows, kv):
    K, r = _inputs(1, H, rows + 5, bits, kv)
    _check(K, r, 3, rows, bits)


@pytest.mark.parametrize("kv", ["bf16", "f32"])
def test_batches(kv):
    K, r = _inputs(3, 5, 4100, 512, kv)
    _check(K[:, :, :4096].contiguous(), r, 1, 4000, 512)


@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("bits", [128, 512])
def test_extreme_values(bits, kv):
    g = torch.Generator().manual_seed(bits)
    rows = 16500
    K, r = _inputs(1, 2, rows, bits, "f32")
    r = r.float()
    K[:, :, 100:300] = 0
    K[:, :, 200:230] = -0.0
    K[:, :, 300:340] = torch.ldexp(torch.randn(K[:, :, 300:340].shape, generator=g), torch.tensor(-100))   # squares underflow
    K[:, :, 340:380] = torch.ldexp(torch.randn(K[:, :, 340:380].shape, generator=g), torch.tensor(-130))
    K[:, :, 400:440] = torch.ldexp(torch.randn(K[:, :, 400:440].shape, generator=g), torch.tensor(120))    # and overflow
    K[:, :, 500:600] = torch.ldexp(K[:, :, 500:600], torch.randint(-60, 60, (1, 2, 100, 128), generator=g))
    K[:, :, 5, 3], K[:, :, 6, 9], K[:, :, 7, 1] = float("nan"), float("inf"), -float("inf")
    r[:, 5:20] = 0
    r[0, 30:40] = torch.ldexp(r[0, 30:40], torch.tensor(-100))
    r[1, 40] = torch.ldexp(r[1, 40], torch.tensor(125))
    r[1, 41, 3] = float("inf")
    _check(K.to(DT[kv]), r.bfloat16(), 0, rows, bits, n_oracle=610, audit=True)


@pytest.mark.parametrize("share", [0.02, 0.5, 1.0])
def test_vectors_that_leave_every_output_open(share):
    """x repeats itself and R repeats itself with the other sign: every sum cancels, no output is settled and the lists
    overflow."""
    g = torch.Generator().manual_seed(2)
    rows, bits = 16500, 256
    K, r = _inputs(1, 2, rows, bits, "bf16")
    r[:, :, 64:] = -r[:, :, :64]
    twice = torch.rand(1, 2, rows, 1, generator=g) < share
    K[..., 64:] = torch.where(twice, K[..., :64], K[..., 64:])
    au = _check(K, r, 0, rows, bits, audit=True)
    assert au["listed"] >= int(twice.sum()) * bits


@pytest.mark.parametrize("kv", ["bf16", "f32"])
def test_zeros_are_settled(kv):
    rows, bits = 16400, 128
    K, r = _inputs(1, 2, rows, bits, kv)
    r[:, 5::3] = -0.0
    zero = torch.zeros_like(K)
    zero[:, :, ::2] = -0.0
    assert _check(zero, r, 0, rows, bits, audit=True)["listed"] == 0
    live = int(r[0].abs().sum(-1).count_nonzero())
    assert _check(K, r, 0, rows, bits, audit=True)["listed"] <= 2 * rows * live // 1000


@pytest.mark.parametrize("kv,open_rows", [("bf16", 1.2e-4), ("f32", 4e-4)])
@pytest.mark.parametrize("factor", [100.0, 1000.0, 1e-14])
def test_rows_of_unequal_norm_have_bounds_of_their_own(factor, kv, open_rows):
    """One row of every word far above the others, or below the norms that count: the other rows are settled as if it were not there
    (equal rows leave 4e-5 of the outputs open, with binary32 vectors 1.3e-4), and of that one at most all outputs are open."""
    rows, bits = 16400, 512
    K, r = _inputs(1, 2, rows, bits, kv)
    W = bits // 32
    r[:, 5 * W:6 * W] = (r[:, 5 * W:6 * W].float() * factor).bfloat16()
    own = 1 / 32 if factor < 1 else 0
    assert _check(K, r, 0, rows, bits, audit=True)["listed"] <= (own + open_rows) * 2 * rows * bits
