"""Register budget of the gfx950 kernels (no GPU needed).

Every kernel source is compiled to device assembly with the library's own
flags, and the code-object metadata of each kernel is read back.  A kernel
that runs out of vector registers spills to scratch memory; inside the
attention loops a spilled value is a memory round trip per tile (a spill of
one uniform value once cost the calibration replay 13% of its time), so the
budget is checked here rather than found in a profile.
"""
import concurrent.futures as cf
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_02029_amd import build

# kernels allowed a little scratch (bytes), each with its reason
SCRATCH_ALLOWED = {
    # one lane offset stored before the tile loop and read back after it
    "replay_attn<256, 8>": 12,
}


def _demangle(name):
    m = re.search(r"(\w+?)I((?:L[ib]-?\d+E)+)E", name)
    if not m:
        return re.sub(r"^_ZN4hwkv12_GLOBAL__N_1\d+", "", name)
    base = re.sub(r"^.*\d", "", re.sub(r"^_ZN4hwkv12_GLOBAL__N_1", "", m.group(1)))
    args = re.findall(r"L[ib](-?\d+)E", m.group(2))   # int and bool arguments
    return f"{base}<{', '.join(args)}>"


def _compile(src, out_dir):
    out = os.path.join(out_dir, os.path.splitext(src)[0] + ".s")
    cmd = [build.HIPCC, *[f for f in build.flags_for(src) if f != "-fPIC"], "--offload-device-only",
           "-S", os.path.join(build.CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out


def _kernels(asm_path):
    """(name, vgpr_count, private_segment_fixed_size) per kernel."""
    text = open(asm_path).read()
    meta = text[text.index("amdhsa.kernels:"):]
    out = []
    for block in re.split(r"\n  - \.", meta)[1:]:
        name = re.search(r"\.name:\s+(\S+)", block)
        vg = re.search(r"\.vgpr_count:\s+(\d+)", block)
        ps = re.search(r"\.private_segment_fixed_size:\s+(\d+)", block)
        if name and vg and ps:
            out.append((_demangle(name.group(1)), int(vg.group(1)), int(ps.group(1))))
    return out


@pytest.fixture(scope="module")
def kernel_table(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not found")
    d = str(tmp_path_factory.mktemp("asm"))
    srcs = [s for s in build.SOURCES if s != "hwkv_api.hip"]
    with cf.ThreadPoolExecutor(max_workers=min(len(srcs), os.cpu_count() or 1)) as ex:
        paths = list(ex.map(lambda s: _compile(s, d), srcs))
    table = {}
    for p in paths:
        for name, vg, ps in _kernels(p):
            table[name] = (vg, ps)
    shutil.rmtree(d, ignore_errors=True)
    return table


def test_every_hot_kernel_is_present(kernel_table):
    for name in ["decode_split<256, 6, 0>", "decode_mfma<256, 6>", "decode_split<256, 6, 1>",
                 "decode_split<256, 8, 0>", "decode_split<64, 1, 0>", "decode_mfma<64, 1>",
                 "decode_mfma<128, 8>",
                 "prefill_attn<256, 8, 0>", "prefill_attn<128, 8, 0>", "prefill_attn<64, 8, 0>",
                 "prefill_attn<256, 8, 1>", "prefill_attn<128, 8, 1>", "prefill_attn<64, 8, 1>",
                 "prefill_merge<256, 8>", "prefill_merge<128, 8>", "prefill_merge<64, 8>",
                 "decode_item<256, 8, 0>", "decode_item<128, 4, 1>", "decode_item<64, 1, 2>",
                 "item_merge<256, 8>", "item_merge<64, 1>",
                 "replay_attn<256, 8>", "replay_merge<256>", "prefill_write<256, 0>",
                 "append_token<256, 2>"]:
        assert name in kernel_table, sorted(kernel_table)


def test_no_scratch_spills(kernel_table):
    bad = {n: ps for n, (vg, ps) in kernel_table.items()
           if ps > SCRATCH_ALLOWED.get(n, 0)}
    assert not bad, f"kernels using scratch memory (bytes): {bad}"


def test_register_budgets(kernel_table):
    # decode splits: four waves per SIMD (128 registers), three (168) for 8 q
    # heads per kv head, whose 64 value accumulators per lane do not fit 128,
    # and for 6 with binary16 keys at head_dim 256; the fp8 matrix-core split
    # and prefill attention: two waves per SIMD (256)
    for n, (vg, _) in kernel_table.items():
        if n.startswith("prefill_attn<") or n.startswith("decode_mfma<"):
            assert vg <= 256, (n, vg)
        if n.startswith("decode_split<"):
            d, g, _f = (int(x) for x in n[n.index("<") + 1:-1].split(","))
            budget = 128
            if g == 8 or (_f == 1 and g == 6 and d >= 256):
                budget = 168
            assert vg <= budget, (n, vg)
        # decode by item: sixteen wavefronts of 128 registers a CU, or eight of 256
        if n.startswith("decode_item<"):
            d, g, _f = (int(x) for x in n[n.index("<") + 1:-1].split(","))
            assert vg <= (256 if g >= 6 or (g == 4 and d == 256) else 128), (n, vg)
