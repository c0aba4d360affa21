"""Prefill attention over fp8 units whose bf16 image is larger than 2^31 bytes:
keys past that mark, in blocks that are not one run of rows (the end of the
cached keys, and a ring's wrap), enter with their values."""
import math

import pytest
import torch

from paper_2609_02029_amd import hwkv

pytestmark = pytest.mark.gpu

D, S, N = 256, 4, 5                    # head_dim, sinks, tokens of the chunk
HALF = 2 ** 30 // D                    # slot at 2^31 bytes of the image
P0 = HALF + 205                        # cached tokens, not a multiple of 32
W = HALF + 40                          # the ring's wrap lies past the mark too
BLOCK = 1 << 18
STEP = 8.0 / 448.0                     # fp8 scale


def _stored(x):
    return (x.float() / STEP).clamp(-448, 448).to(torch.float8_e4m3fn).float() * STEP


# `loud`: the cached positions [lo, hi) whose keys point along the query and
# whose values are 1, so that they carry about half of the weights
@pytest.mark.parametrize("window,loud", [(0, (P0 - 13, P0)), (W, (S + W - 17, S + W)),
                                         (W, (S + W, S + W + 15)), (W, (P0 - 13, P0))])
def test_keys_past_the_mark(window, loud):
    gen = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    pol = hwkv.policy_set(1, 1, 1, D, S, [window], [[0]])
    cache = hwkv.cache_alloc(pol, 1, P0 + N + 64, kv_format="fp8", k_scale=STEP, v_scale=STEP)
    q1 = rnd(1, 1, D)
    kb, vb = rnd(BLOCK, 1, D), rnd(BLOCK, 1, D)
    scale = 1.0 / math.sqrt(D)
    # each loud key's logit: log(weight of the others / how many there are)
    far = math.log(P0 * math.exp(0.5) / (loud[1] - loud[0]))
    key = (q1.float() * (far / (scale * float(q1.float().pow(2).sum())))).to(torch.bfloat16)
    one = torch.ones(1, 1, D, device="cuda", dtype=torch.bfloat16)
    pieces = []                        # (first position, keys, values), as cached
    for a in range(0, P0, BLOCK):
        b = min(P0, a + BLOCK)
        k, v = kb[:b - a], vb[:b - a]
        lo, hi = max(a, loud[0]), min(b, loud[1])
        if lo < hi:
            k, v = k.clone(), v.clone()
            k[lo - a:hi - a], v[lo - a:hi - a] = key, one
        pieces.append((a, k, v))
        hwkv.prefill_write(cache, 0, 0, a, k, v)
    k, v, q = rnd(N, 1, D), rnd(N, 1, D), q1.expand(N, 1, D).contiguous()
    ws = torch.empty(hwkv.prefill_attn_workspace_bytes(cache, N), dtype=torch.uint8, device="cuda")
    out = torch.empty(N, 1, D, device="cuda")
    hwkv.prefill_attn(cache, 0, 0, P0, q, k, v, scale, out, ws=ws)
    cache.free()

    w1, wv = torch.zeros(N, 1, device="cuda"), torch.zeros(N, D, device="cuda")
    pos = P0 + torch.arange(N, device="cuda")[:, None]
    for a, kp, vp in pieces + [(P0, k, v)]:
        at = a + torch.arange(len(kp), device="cuda")[None, :]
        seen = at <= pos
        if window:
            seen &= (at < S) | (at > pos - window)
        z = _stored(kp[:, 0]) @ q1[0, 0].float() * scale
        p = torch.where(seen, torch.exp(z)[None, :], 0.0)
        w1 += p.sum(1, keepdim=True)
        wv += p @ _stored(vp[:, 0])
    ref = wv / w1
    share = float(ref[-1].mean())
    assert 0.2 < share < 0.8           # the loud values' share of the weights
    # weights are rounded to bf16 (2^-9 each); the loud ones dominate the sum
    assert float((out[:, 0] - ref).abs().max()) <= 2 ** -8
