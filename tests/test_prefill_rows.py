"""Row addresses of prefill attention's key-by-key loads (no GPU needed): the
kernel's own arithmetic, compiled for the host, against the cache layout in 64
bits, over units up to the largest an allocation takes."""
import ctypes
import shutil
import subprocess

import pytest

from paper_2609_02029_amd import build

SOURCE = """
#include "hwkv_internal.h"
extern "C" void rows(int D, int s0, int S, int W, uint32_t *k, uint32_t *v) {
  for (int i = 0; i < 32; ++i) {
    const int slot = hwkv::cached_slot(s0 + i, S, W);
    k[i] = hwkv::cached_k(D, slot);
    v[i] = hwkv::cached_v(D, slot);
  }
}
extern "C" uint32_t span() { return hwkv::kRowSpan; }
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    if not shutil.which(build.HIPCC):
        pytest.skip("hipcc not found")
    d = tmp_path_factory.mktemp("rows")
    (d / "rows.hip").write_text(SOURCE)
    subprocess.run([build.HIPCC, *build.CFLAGS, "-O1", "--offload-host-only", "-shared",
                    str(d / "rows.hip"), "-o", str(d / "rows.so")], check=True, capture_output=True)
    lib = ctypes.CDLL(str(d / "rows.so"))
    lib.span.restype = ctypes.c_uint32

    def call(D, s0, S, W):
        out = [(ctypes.c_uint32 * 32)() for _ in range(2)]
        lib.rows(D, s0, S, W, *out)
        return [list(x) for x in out]

    call.span = lib.span()
    return call


def layout(D, slot):
    """Byte offsets of a slot's first K chunk and of its V row (2-byte elements)."""
    return slot // 64 * (64 * D * 2) + slot % 64 * 16, slot * D * 2


@pytest.mark.parametrize("D", [64, 128, 256])
def test_offsets_at_any_slot(rows, D):
    top = (2 ** 31 - 1) // D // 64 * 64               # slots of the largest fp8 unit
    half = 2 ** 30 // D                               # its 2^31-byte mark as bf16
    assert 2 ** 31 < top * D * 2 <= rows.span
    for S, W in [(0, 0), (4, 0), (0, half + 1), (33, top - 40), (4, 500), (3, 1), (0, 31), (70, 33)]:
        cap = S + W if W else top
        starts = {0, 1, 32, S, max(0, S - 31), half - 32, half - 16, half, half + 32, cap - 40, cap - 32, cap - 5,
                  cap, cap + half // 2}
        for s0 in sorted(starts):
            if s0 < 0 or s0 + 32 > (top if W == 0 else 2 * top):
                continue
            k, v = rows(D, s0, S, W)
            for i in range(32):
                s = s0 + i
                slot = s if W == 0 or s < S else S + (s - S) % W
                assert (k[i], v[i]) == layout(D, slot), (S, W, s0, i)
                # the last loads of the row stay within the descriptor's span
                assert k[i] + (D // 8 - 1) * 1024 + 16 <= rows.span and v[i] + D * 2 <= rows.span
