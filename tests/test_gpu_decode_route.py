"""Which kernels a decode batch runs on -- split workgroups and a merge for every
64 items, or a workgroup per item, its long items split and merged -- and parity
on each side: the launch counts and merge times that the library's own timing
reports say which one ran."""
import numpy as np
import pytest
import torch

from hwkv_harness import Run
from paper_2609_02029_amd import hwkv
from test_gpu_formats import fmt_args, mini

pytestmark = pytest.mark.gpu


def _route(r, fused):
    """One checked step; (launches, whether one of them was merged)."""
    hwkv.decode_timing(r.cache, True)
    qa, out = r.step(0, fused=fused)
    torch.cuda.synchronize()
    _, merge_ms, launches = hwkv.decode_timing_read(r.cache)
    hwkv.decode_timing(r.cache, False)
    r.check_out(0, qa, out, f"fused={fused}")
    return launches, merge_ms > 0.0


def _run(cfg, pages=False, **kw):
    """Checks two steps and the residency; their routes."""
    n_pages = sum(-(-(n + 2) // 256) for n in cfg["prompt"]) * sum(
        1 for h in cfg["levels"][0] if cfg["level_windows"][h] == 0) if pages else None
    r = Run(cfg, n_pages=n_pages, **kw)
    for b in range(r.B):
        r.prefill(0, b)
    routes = {_route(r, fused) for fused in (True, False)}
    r.check_layer(0)
    r.free()
    return routes


# 72 sequences x 2 heads (one windowed) with some of 2,000 to 4,100 tokens: the
# full head's long items are split in up to five; the appended tokens of the
# fused step go to the first, a middle or the last split (and, in the windowed
# head, anywhere in the ring)
RAGGED = [4099, 4096, 3071, 3072, 2111, 2048, 1343, 1344] + [33 + 29 * i % 600 for i in range(64)]


@pytest.mark.parametrize("fmt,D,G,paged", [
    ("bf16", 64, 1, False), ("bf16", 128, 4, False), ("bf16", 64, 8, True), ("f16", 128, 2, True),
    ("f16", 64, 6, False), ("fp8", 64, 1, False), ("fp8", 64, 4, True), ("bf16", 256, 4, False)])
def test_split_items_and_their_merge(fmt, D, G, paged):
    cfg = mini(head_dim=D, n_q_heads=4 * G, n_kv_heads=4, batch=len(RAGGED), n_sinks=3,
               level_windows=[1555, 0], levels=[[0, 1, 0, 0]], prompt=RAGGED, max_ctx=4200, seed=81)
    assert _run(cfg, paged, **fmt_args(fmt, 0.013, 0.009, 1, 4)) == {(1, True)}


# Each head_dim, group and format on whole items: enough short ones for every
# group (96 x 8 of one to four tiles)
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("G", [1, 2, 4, 6, 8])
@pytest.mark.parametrize("fmt", ["bf16", "f16", "fp8"])
def test_whole_items_of_every_kind(D, G, fmt):
    n = [1 + 41 * i % 250 for i in range(96)]
    cfg = mini(head_dim=D, n_q_heads=8 * G, n_kv_heads=8, batch=96, n_sinks=2, level_windows=[47, 0],
               levels=[[0, 1, 0, 1, 1, 0, 0, 0]], prompt=n, max_ctx=260, seed=82)
    assert _run(cfg, **fmt_args(fmt, 0.013, 0.009, 1, 8)) == {(1, False)}


# Batches that run split in more than one launch group: partials and page
# offsets of the second group
@pytest.mark.parametrize("fmt,paged", [("bf16", False), ("bf16", True), ("f16", True), ("fp8", False),
                                       ("fp8", True)])
def test_split_launch_groups(fmt, paged):
    cfg = mini(head_dim=256, n_q_heads=32, n_kv_heads=4, batch=17, n_sinks=4, level_windows=[900, 0],
               levels=[[1, 0, 1, 0]], prompt=[1010 + 5 * i for i in range(17)], max_ctx=1200, seed=83)
    assert _run(cfg, paged, **fmt_args(fmt, 0.013, 0.009, 1, 4)) == {(2, True)}
