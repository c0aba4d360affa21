"""Prefill attention whose keys are split over workgroups (few query tokens
over many keys): parity at the edges of tiles, runs and splits, and the split
partials -- a captured call without a buffer for them (which runs unsplit) and
with one, calls on several streams, and no memory held after a call."""
import numpy as np
import pytest
import torch

from hwkv_harness import Run
from paper_2609_02029_amd import hwkv
from test_gpu_formats import _check_stored_rows, fmt_args
from test_gpu_prefill_attn import check_rows, mini

pytestmark = pytest.mark.gpu


# windows around the 32- and 64-key blocks and the ring's wrap, page and tile
# edges, chunks of one token and of a ragged 32-column block
@pytest.mark.parametrize("fmt,paged", [("bf16", False), ("bf16", True), ("f16", True), ("fp8", False)])
@pytest.mark.parametrize("D,G,S,windows,cuts", [
    (64, 1, 0, [63, 1000, 0], [1500, 3000, 3001]),
    (128, 8, 4, [64, 1111, 0], [2048, 3040, 3072]),
    (256, 6, 33, [31, 1984, 0], [2047, 3071, 3072]),
    (128, 4, 5, [2500, 97, 0], [2560, 2900]),
])
def test_few_tokens_over_many_keys(fmt, paged, D, G, S, windows, cuts):
    P = 3110
    cfg = mini(head_dim=D, n_q_heads=3 * G, n_kv_heads=3, n_sinks=S, level_windows=windows,
               levels=[[0, 1, 2]], prompt=[P], max_ctx=P + 10, seed=51)
    r = Run(cfg, n_pages=14 if paged else None, **fmt_args(fmt, 0.013, 0.009, 1, 3))
    q, qh, out = r.prefill_with_attn(0, 0, chunks=cuts)
    near = [t + d for t in cuts + [S, P] for d in range(-3, 3)]
    rows = np.unique([t for t in near + list(range(0, P, 97)) if 0 <= t < P])
    if fmt == "bf16":
        check_rows(r, 0, 0, rows, qh[rows], out, f"D={D} {windows}")
    else:
        _check_stored_rows(r, 0, 0, rows, qh[rows], out, f"{fmt} D={D} {windows}")
    r.check_layer(0)
    r.free()


# launches of one to three key tiles (without and with the phase shift), whose
# tiles are all partly visible: chunks that end at, before and past the edges
# of a mask's word, a tile and a block of columns
@pytest.mark.parametrize("D,G,S,windows", [
    (64, 1, 0, [1, 33, 0]), (128, 2, 31, [32, 64, 0]), (256, 6, 1, [30, 65, 0]),
])
def test_few_keys(D, G, S, windows):
    cuts = [1, 2, 32, 63, 65, 97, 128, 160]
    cfg = mini(head_dim=D, n_q_heads=3 * G, n_kv_heads=3, n_sinks=S, level_windows=windows,
               levels=[[0, 1, 2]], prompt=[193], max_ctx=200, seed=53)
    r = Run(cfg)
    q, qh, out = r.prefill_with_attn(0, 0, chunks=cuts)
    check_rows(r, 0, 0, np.arange(193), qh, out, f"D={D} {windows}")
    r.check_layer(0)
    r.free()


def _pair(seed):
    """Two sequences of 4,000 cached tokens, and a 40-token chunk of each."""
    cfg = mini(batch=2, head_dim=128, n_q_heads=8, level_windows=[700, 0], prompt=[4000, 4000],
               max_ctx=4100, seed=seed)
    r = Run(cfg)
    g = torch.Generator(device="cuda").manual_seed(seed)
    for b in range(2):
        r.prefill(0, b)
    x = lambda h: torch.randn((40, h, 128), generator=g, device="cuda").to(torch.bfloat16)
    return r, [(x(8), x(2), x(2)) for _ in range(2)]


def test_captured_call_runs_unsplit_and_replays():
    r, ((q, k, v), _) = _pair(61)
    eager, captured = torch.empty(2, 40, 8, 128, device="cuda")
    call = lambda out: hwkv.prefill_attn(r.cache, 0, 0, 4000, q, k, v, r.scale, out)
    call(eager)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(captured)
    for i in range(3):
        captured.fill_(float("nan"))
        g.replay()
        again = torch.empty_like(eager)
        call(again)                       # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(again, eager)
        # another order of the sums, and of the weights' rounding to bf16
        assert not torch.equal(captured, eager)
        bound = (2 * 2.0 ** -8 + 4e-5) * 8.0   # twice the weight-rounding bound, |v| < 8
        assert float((captured - eager).abs().max()) <= bound
    r.free()


def test_captured_call_with_parts_splits():
    r, ((q, k, v), _) = _pair(63)
    out = torch.empty(2, 40, 8, 128, device="cuda")
    nbytes = hwkv.prefill_attn_split_bytes(r.cache, 0, 4000, 40)
    assert nbytes > 0
    parts = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    call = lambda o, p: hwkv.prefill_attn(r.cache, 0, 0, 4000, q, k, v, r.scale, o, parts=p)
    call(out[0], None)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(out[1], parts)
    for i in range(3):
        parts.fill_(255)                  # NaN
        out[1].fill_(float("nan"))
        g.replay()
        call(out[0], None)
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[1])
    # too small a buffer: unsplit, as without one
    small = torch.empty(2, 40, 8, 128, device="cuda")
    call(small[0], parts[:nbytes - 16])
    h = torch.cuda.CUDAGraph()
    with torch.cuda.graph(h):
        call(small[1], None)
    h.replay()
    torch.cuda.synchronize()
    assert torch.equal(small[0], small[1]) and not torch.equal(small[0], out[0])
    r.free()


def _held():
    """Device memory in use beside torch's own pool."""
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free - torch.cuda.memory_reserved()


def test_a_split_call_keeps_no_memory():
    r, chunks = _pair(64)
    (q, k, v), _ = chunks
    out = torch.empty(40, 8, 128, device="cuda")
    g = torch.cuda.CUDAGraph()            # the kernels are loaded, none has split
    with torch.cuda.graph(g):
        hwkv.prefill_attn(r.cache, 0, 0, 4000, q, k, v, r.scale, out)
    g.replay()
    streams = [torch.cuda.Stream() for _ in range(3)]
    for s in streams:                     # their queues are made
        with torch.cuda.stream(s):
            torch.zeros(1 << 20, device="cuda")
    before, used = _held(), torch.cuda.memory_allocated()
    for s in (None, streams[0], streams[1], streams[2].cuda_stream):
        hwkv.prefill_attn(r.cache, 0, 0, 4000, q, k, v, r.scale, out, stream=s)
    assert _held() - before < (1 << 22)
    assert torch.cuda.memory_allocated() == used
    r.free()


# Calls of four streams in flight at once, over caches of two head dims (partials
# of two sizes): each has the result of a call alone.
def test_many_streams_at_once():
    jobs = []
    for D, seed in ((64, 65), (256, 66), (64, 67), (256, 68)):
        cfg = mini(head_dim=D, n_q_heads=8, level_windows=[700, 0], prompt=[6000], max_ctx=6100, seed=seed)
        r = Run(cfg)
        r.prefill(0, 0)
        g = torch.Generator(device="cuda").manual_seed(seed)
        x = lambda h: torch.randn((40, h, D), generator=g, device="cuda").to(torch.bfloat16)
        args = (r.cache, 0, 0, 6000, x(8), x(2), x(2), r.scale)
        assert hwkv.prefill_attn_split_bytes(r.cache, 0, 6000, 40) > 0
        lone = torch.empty(40, 8, D, device="cuda")
        hwkv.prefill_attn(*args, lone)
        torch.cuda.synchronize()
        jobs.append((r, args, lone, torch.cuda.Stream(),
                     [torch.full_like(lone, float("nan")) for _ in range(12)]))
    torch.cuda.synchronize()
    for i in range(12):
        for r, args, lone, stream, outs in jobs:
            hwkv.prefill_attn(*args, outs[i], stream=stream)
    torch.cuda.synchronize()
    for r, args, lone, stream, outs in jobs:
        assert all(torch.equal(o, lone) for o in outs)
        r.free()


def test_two_streams_of_one_cache():
    r, chunks = _pair(62)
    lone = []
    for b, (q, k, v) in enumerate(chunks):
        lone.append(torch.empty(40, 8, 128, device="cuda"))
        hwkv.prefill_attn(r.cache, 0, b, 4000, q, k, v, r.scale, lone[b])
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[torch.full((40, 8, 128), float("nan"), device="cuda") for _ in range(2)]
            for _ in range(8)]
    torch.cuda.synchronize()
    for o in outs:
        for b, (q, k, v) in enumerate(chunks):
            hwkv.prefill_attn(r.cache, 0, b, 4000, q, k, v, r.scale, o[b], stream=streams[b])
    torch.cuda.synchronize()
    for o in outs:
        assert torch.equal(o[0], lone[0]) and torch.equal(o[1], lone[1])
    r.free()
