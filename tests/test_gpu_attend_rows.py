"""Sparse attention at the row counts where its row tile changes and where a workgroup takes a head whole,
for few and many heads, both element types, with duplicates and indices outside the cache: against
the oracle (binary64).  Tolerance: binary32 sums of at most 520 terms and exp to a few units in the last
place, relative to outputs of order 1: 520 * 2^-24 + 1e-6 < 4e-5."""
import math

import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,Hq,Hkv", [(1, 3, 3), (4, 32, 8)])
@pytest.mark.parametrize("k", [1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 511, 512, 513])
def test_row_counts(B, Hq, Hkv, k, kv):
    import paper_2508_19740_amd as sp
    g = torch.Generator().manual_seed(k + Hq)
    n = 700
    q, K, V = (torch.randn(*s, generator=g).to(kv) for s in ((B, Hq, 128), (B, Hkv, n, 128), (B, Hkv, n, 128)))
    idx = torch.randint(0, n, (B, Hq, k), generator=g, dtype=torch.int32)      # any order, duplicates count twice
    if k > 4:
        idx[:, :, 3], idx[:, :, k - 1] = -1, n                                 # skipped
    scale = 1.0 / math.sqrt(128)
    dev = torch.device("cuda:0")
    ctx = sp.Spotlight(B, Hq, Hkv, 64, 0, n, k, kv_dtype=kv, device=dev)
    try:
        got = ctx.sparse_decode(q.to(dev), K.to(dev), V.to(dev), idx.to(dev), scale).cpu()
        ran = None
        ctx.profile_enable(True)
        again = ctx.sparse_decode(q.to(dev), K.to(dev), V.to(dev), idx.to(dev), scale).cpu()
        ran = ctx.profile_read()
        assert ran["attend"][1] == ran["merge"][1] == 1                        # the merge counts as a stage wherever it runs
    finally:
        ctx.close()
    assert torch.equal(got, again)
    rep = Hq // Hkv
    kept = ((idx >= 0) & (idx < n))
    at = idx.clamp(0, n - 1).long().unsqueeze(-1).expand(-1, -1, -1, 128)
    Kg = K.double().repeat_interleave(rep, 1).gather(2, at)
    Vg = V.double().repeat_interleave(rep, 1).gather(2, at)
    s = (Kg * q.double().unsqueeze(2)).sum(-1) * scale
    p = torch.softmax(s.masked_fill(~kept, float("-inf")), -1)
    want = (p.unsqueeze(-1) * Vg).sum(2)
    assert float((got.double() - want).abs().max()) < 4e-5
    if k <= 4:
        assert float((got - oracle.sparse_decode(q, K, V, idx, scale)).abs().max()) < 4e-5
