"""One-vector hashing from the packed copy of the weights where the width of a workgroup changes (more than
512 hidden units, bfloat16 weights, at most a vector per compute unit): appended code and selected
indices equal the oracle's and those hashed from the arrays as stored."""
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv", [(1, 2, 2), (16, 16, 8)])                 # 4 and 384 vectors a step
@pytest.mark.parametrize("kv", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("w", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("bits,hidden", [(256, 512), (512, 640), (32, 896), (160, 1024), (512, 1152)])
def test_packed_widths(bits, hidden, w, kv, B, Hq, Hkv):
    import paper_2508_19740_amd as sp
    g = torch.Generator().manual_seed(bits + hidden)
    dev, n, k = torch.device("cuda:0"), 40, 7
    q, K, V = (torch.randn(*s, generator=g).to(kv) for s in ((B, Hq, 128), (B, Hkv, n, 128), (B, Hkv, n, 128)))
    ws = [(0.05 * torch.randn(Hkv, *s, generator=g)).to(w) for s in ((hidden, 128), (hidden,), (bits, hidden))]
    codes = torch.randint(-2**31, 2**31 - 1, (B, Hkv, n, bits // 32), generator=g, dtype=torch.int32)
    got = []
    for packed in (False, True):
        ctx = sp.Spotlight(B, Hq, Hkv, bits, hidden, n, k, kv_dtype=kv, weight_dtype=w, device=dev)
        try:
            on = [t.to(dev) for t in ws]
            if packed:
                ctx.prepack_weights(*on)
            c = codes.to(dev)
            idx, _ = ctx.decode_step(q.to(dev), K.to(dev), V.to(dev), *on, c, n, k)
            got.append((c.cpu(), idx.cpu()))
        finally:
            ctx.close()
    want = codes.clone()
    oracle.hash_keys(K, *ws, bits, n - 1, 1, want)
    assert torch.equal(got[0][0], want) and torch.equal(got[1][0], want)
    assert torch.equal(got[0][1], got[1][1])
