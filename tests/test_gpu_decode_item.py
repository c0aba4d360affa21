"""Decode with a workgroup per (sequence, KV head) item (batches of many short
items): parity over head dims, groups and formats at the edges of tiles, of a
workgroup's waves and of the windows, and over more sequences than one launch
takes."""
import numpy as np
import pytest
import torch

from hwkv_harness import Run
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
