"""The score kernel's workgroup widths at the edges of their dispatch: grids of at most one block per
compute unit (1024 threads), grids just above, and long runs of blocks, for every group size and for code
lengths of each lane split; candidate sub-lists that overflow (k near the number of tokens) and
windows that fill the tokens of a thread.  Indices equal the oracle's on the codes of the cache."""
import pytest
import torch

import oracle
import workload as wl

pytestmark = pytest.mark.gpu


def _check(B, Hkv, G, n, bits, k, n_sink=0, n_local=0, heads=3, seed=5):
    import paper_2508_19740_amd as sp
    cfg = wl.CONFIGS["C2"].scaled(batch=B, n_q_heads=Hkv * G, n_kv_heads=Hkv, n_tokens=n, code_bits=bits, hidden=0, topk=k, needles=0,
                                  seed=seed + n)
    dev = torch.device("cuda:0")
    w = wl.Workload(cfg)
    q, weights = w.q.to(dev), [None if t is None else t.to(dev) for t in w.hash_weights()]
    codes = torch.empty(B, Hkv, n, bits // 32, dtype=torch.int32, device=dev)
    for b in range(B):
        for h in range(Hkv):
            codes[b, h] = w.synthetic_codes(b, h, 0, n, dev)
    K = torch.randn(B, Hkv, n, 128, device=dev).bfloat16()
    ctx = sp.Spotlight(B, Hkv * G, Hkv, bits, 0, n, k, device=dev)
    try:
        idx, _ = ctx.decode_step(q, K, K, *weights, codes, n, k, n_sink, n_local)
        torch.cuda.synchronize()
        idx, codes = idx.cpu(), codes.cpu()
    finally:
        ctx.close()
    hw = w.hash_weights()
    for i in range(heads):   # the first, the last and one in between: heads are independent
        bh = i * (B * Hkv - 1) // max(1, heads - 1)
        b, h = bh // Hkv, bh % Hkv
        sub = (w.q[b:b + 1, h * G:(h + 1) * G].contiguous(), *[None if t is None else t[h:h + 1].contiguous() for t in hw])
        want = oracle.decode_step(sub[0], K[b:b + 1, h:h + 1].cpu(), K[b:b + 1, h:h + 1].cpu(), *sub[1:], codes[b:b + 1, h:h + 1].contiguous(),
                                  n, k, n_sink, n_local, 128 ** -0.5)[0]
        assert torch.equal(idx[b:b + 1, h * G:(h + 1) * G], want), (b, h)


@pytest.mark.parametrize("G", range(1, 9))
@pytest.mark.parametrize("bits", [32, 96, 128, 256, 512])
def test_small_grid(G, bits):
    _check(1, 2, G, 4096 + 77, bits, 90)


@pytest.mark.parametrize("G,bits", [(1, 128), (2, 64), (2, 128), (3, 128), (4, 256), (4, 512), (5, 64), (7, 128), (8, 256), (8, 512)])
def test_more_blocks_than_compute_units(G, bits):
    _check(2, 44, G, 3 * 4096 - 5, bits, 150, 4, 64)       # 264 blocks


@pytest.mark.parametrize("G,bits", [(1, 32), (4, 96), (8, 32)])
def test_runs_of_several_blocks(G, bits):
    _check(32, 16, G, 5 * 4096 + 1, bits, 400, 0, 1, heads=2)      # 3072 blocks


@pytest.mark.parametrize("k", [1, 700, 1500, 2100, 2170])
@pytest.mark.parametrize("G", [1, 8])
def test_sub_lists_that_overflow(G, k):
    _check(1, 1, G, 2170, 128, k, heads=1)


@pytest.mark.parametrize("n_sink,n_local", [(0, 64), (8, 300), (64, 0), (0, 9)])
@pytest.mark.parametrize("B", [1, 300])
def test_windows_that_fill_a_threads_tokens(B, n_sink, n_local):
    _check(B, 8 if B > 1 else 1, 4, 4096 + 640, 64, 400, n_sink, n_local, heads=2)   # both select widths


# the code lengths and groups on either side of every line of the rule that gives a score workgroup its threads
# and registers: 1024 threads or 512 with 256 registers up to a block per compute unit, 512 with 128 up to two, by
# generations above (two of either width between three and four blocks; four and three from six on)
@pytest.mark.parametrize("Hkv,B", [(5, 4), (25, 6), (28, 10), (40, 11), (40, 20)])     # 40, 300, 560, 880 and 1600 blocks
@pytest.mark.parametrize("bits,G", [(32, 3), (64, 6), (64, 7), (128, 3), (128, 4), (160, 4), (192, 8), (224, 7), (224, 8), (256, 6), (256, 7),
                                    (288, 6), (288, 7), (320, 5), (320, 6), (352, 3), (352, 4), (352, 5), (384, 2), (384, 3), (416, 1), (416, 2),
                                    (416, 3), (416, 8), (448, 1), (448, 2), (448, 8), (480, 1), (480, 2), (480, 3), (480, 8), (512, 4),
                                    (512, 5), (512, 8), (1024, 1), (1024, 2)])
def test_widths_by_registers(bits, G, Hkv, B):
    _check(B, Hkv, G, 4096 + 50, bits, 60, 2, 3, heads=2)


@pytest.mark.parametrize("B", [6, 12])     # 300 and 600 blocks: the widths above a block per compute unit
@pytest.mark.parametrize("words,G", [(w, g) for w in list(range(1, 17)) + [32] for g in range(1, 9) if not (w == 32 and g > 2)])
def test_every_pair_on_larger_grids(words, G, B):
    _check(B, 25, G, 4096 + 9 + words, words * 32, 50, 1, 2, heads=1)
