"""Decode with a workgroup per (sequence, KV head) item (batches of many short
items): parity over head dims, groups and formats at the edges of tiles, of a
workgroup's waves and of the windows, and over more sequences than one launch
takes.  (test_gpu_decode_route.py checks which batches run by
item, and their long items.)"""
import numpy as np
import pytest
import torch

from hwkv_harness import Run
from paper_2609_02029_amd import hwkv
from test_gpu_formats import fmt_args, mini

pytestmark = pytest.mark.gpu


def _check(cfg, steps=2, **kw):
    r = Run(cfg, **kw)
    for b in range(r.B):
        r.prefill(0, b)
    for st in range(steps):
        qa, out = r.step(0, fused=st % 2 == 0)
        r.check_out(0, qa, out, f"step {st}")
    r.check_layer(0)
    r.free()


# 70 sequences of one to 1,090 tokens: lengths at the edges of the 64-slot
# tiles, of 8 and 16 tiles (one for every wave), and past them
LENGTHS = ([1, 2, 62, 63, 64, 65, 127, 128, 510, 511, 512, 513, 575, 1022, 1023, 1024, 1025, 1089]
           + [1 + 37 * i % 700 for i in range(52)])


@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("G", [1, 2, 4, 6, 8])
@pytest.mark.parametrize("fmt", ["bf16", "f16", "fp8"])
def test_many_short_items(D, G, fmt):
    cfg = mini(head_dim=D, n_q_heads=2 * G, batch=70, n_sinks=3, level_windows=[61, 0],
               levels=[[0, 1]], prompt=LENGTHS, max_ctx=1100, seed=71)
    _check(cfg, **fmt_args(fmt, 0.013, 0.009, 1, 2))


@pytest.mark.parametrize("fmt", ["bf16", "fp8"])
def test_paged_items(fmt):
    cfg = mini(head_dim=128, n_q_heads=8, batch=70, n_sinks=0, level_windows=[256, 0],
               levels=[[0, 1]], prompt=LENGTHS, max_ctx=1100, seed=72)
    pages = sum(-(-(n + 2) // 256) for n in LENGTHS)
    _check(cfg, n_pages=pages, **fmt_args(fmt, 0.013, 0.009, 1, 2))


def test_more_sequences_than_one_launch():
    n = [1 + i % 90 for i in range(300)]
    cfg = mini(head_dim=64, n_q_heads=4, n_kv_heads=1, batch=300, n_sinks=2, level_windows=[40, 0],
               levels=[[1]], prompt=n, max_ctx=100, seed=73)
    _check(cfg)


# A head's logit is the sum of four partial ones.  One channel of every key makes
# 2^12 of it, and the other pairs of channels of every second key less than half
# an ulp of that (2^-12) each: a partial logit that holds the large product
# loses them all, the three others keep theirs, so at most a quarter of their sum
# is lost.
@pytest.mark.parametrize("D,G", [(64, 4), (128, 1), (128, 4), (256, 2)])
@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("big", [0, -1])
def test_small_products_beside_a_large_one(D, G, fmt, big):
    B, H, n = 64, 4, 512
    pol = hwkv.policy_set(1, H, H * G, D, 0, [0], [[0] * H])
    cache = hwkv.cache_alloc(pol, B, n + 8, kv_format=fmt)
    small = 1.40625 * 2.0 ** -14
    k = torch.zeros(n, H, D, device="cuda")
    k[1::2] = small
    k[:, :, 0:2 if big == 0 else 0] = 0.0
    k[:, :, D - 2 if big else D:] = 0.0
    k[:, :, big] = 64.0
    q = torch.ones(B, H * G, D, device="cuda")
    q[:, :, big] = 64.0
    v = torch.zeros(n, H, D, device="cuda")
    v[1::2] = 1.0
    k, v, q = (x.to(torch.bfloat16) for x in (k, v, q))
    for b in range(B):
        hwkv.prefill_write(cache, 0, b, 0, k, v)
    out = torch.empty(B, H * G, D, device="cuda")
    ws = torch.empty(hwkv.decode_workspace_bytes(cache), dtype=torch.uint8, device="cuda")
    hwkv.decode_timing(cache, True)
    hwkv.decode_attn(cache, 0, q, 1.0, out, ws)
    torch.cuda.synchronize()
    assert hwkv.decode_timing_read(cache)[2] == 1     # by item: one launch for 256 items
    hwkv.decode_timing(cache, False)
    cache.free()
    delta = (D - 2) * small                           # exact difference of the logits
    lost = (D // 4) * small                           # a quarter's
    ulp = 5 * 2.0 ** -12                              # of 2^12: three sums and the scaling of two logits
    ref = 1.0 / (1.0 + np.exp(-delta))
    assert float((out - ref).abs().max()) <= 0.25 * (lost + ulp)
    assert 0.25 * (delta - lost - ulp) > 0.25 * (lost + ulp)   # all of them lost would show


# Tiles whose logits are all -inf (infinite keys) weigh nothing, wherever a wave
# meets them.
@pytest.mark.parametrize("D,G,fmt", [(64, 1, "bf16"), (128, 4, "bf16"), (256, 8, "f16")])
@pytest.mark.parametrize("lo,hi", [(0, 64), (64, 128), (128, 512), (320, 448)])
def test_tiles_of_minus_infinity(D, G, fmt, lo, hi):
    B, H, n = 64, 4, 512
    gen = torch.Generator(device="cuda").manual_seed(9)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    pol = hwkv.policy_set(1, H, H * G, D, 0, [0], [[0] * H])
    cache = hwkv.cache_alloc(pol, B, n + 8, kv_format=fmt)
    k, v, q = rnd(n, H, D), rnd(n, H, D), rnd(B, H * G, D)
    q[:, :, 0] = -1.0
    k[lo:hi, :, 0] = float("inf")
    for b in range(B):
        hwkv.prefill_write(cache, 0, b, 0, k, v)
    out = torch.empty(B, H * G, D, device="cuda")
    ws = torch.empty(hwkv.decode_workspace_bytes(cache), dtype=torch.uint8, device="cuda")
    hwkv.decode_timing(cache, True)
    hwkv.decode_attn(cache, 0, q, 0.1, out, ws)
    torch.cuda.synchronize()
    assert hwkv.decode_timing_read(cache)[2] == 1     # by item
    cache.free()
    keep = torch.tensor([i for i in range(n) if not lo <= i < hi], device="cuda")
    as64 = (lambda x: x.to(torch.float16).double()) if fmt == "f16" else (lambda x: x.double())
    kk, vv = as64(k[keep]).permute(1, 2, 0).contiguous(), as64(v[keep]).permute(1, 0, 2).contiguous()
    z = torch.matmul(q.double().reshape(B, H, G, D), kk) * 0.1
    ref = torch.matmul(torch.softmax(z, -1), vv).reshape(B, H * G, D)
    assert float((out - ref).abs().max()) <= 2e-5 * 8.0   # fp32 sums, |v| < 8
