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
extern "C" void rows(int D, int s0, int S, int W, int paged, int64_t *k, int64_t *v, int64_t *at) {
  const int first = paged ? s0 % hwkv::kPageTokens : hwkv::cached_slot(s0, S, W);
  for (int i = 0; i < 32; ++i) {
    const int slot = paged ? first + i : hwkv::cached_slot(s0 + i, S, W);
    const hwkv::CachedRow r = hwkv::cached_row(D, slot, first, S);
    k[i] = hwkv::cached_base_k(D, r.base) + r.k;
    v[i] = hwkv::cached_base_v(D, r.base) + r.v;
    at[i] = r.k < r.v ? r.v : r.k;
    if (r.k < 0 || r.v < 0) at[i] = -1;
  }
}
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

    def call(D, s0, S, W, paged=0):
        out = [(ctypes.c_int64 * 32)() for _ in range(3)]
        lib.rows(D, s0, S, W, paged, *out)
        return [list(x) for x in out]

    return call


def layout(D, slot):
    """Byte offsets of a slot's first K chunk and of its V row (2-byte elements)."""
    return slot // 64 * (64 * D * 2) + slot % 64 * 16, slot * D * 2


@pytest.mark.parametrize("D", [64, 128, 256])
def test_offsets_at_any_slot(rows, D):
    top = (2 ** 31 - 1) // D // 64 * 64               # slots of the largest fp8 unit
    half = 2 ** 30 // D                               # its 2^31-byte mark as bf16
    assert top * D * 2 > 2 ** 31
    for S, W in [(0, 0), (4, 0), (0, half + 1), (33, top - 40), (4, 500), (3, 1), (0, 31), (70, 33)]:
        cap = S + W if W else top
        starts = {0, 1, 32, S, max(0, S - 31), half - 32, half - 16, half, half + 32, cap - 40, cap - 32, cap - 5,
                  cap, cap + half // 2}
        for s0 in sorted(starts):
            if s0 < 0 or s0 + 32 > (top if W == 0 else 2 * top):
                continue
            k, v, at = rows(D, s0, S, W)
            for i in range(32):
                s = s0 + i
                slot = s if W == 0 or s < S else S + (s - S) % W
                assert (k[i], v[i]) == layout(D, slot), (S, W, s0, i)
                # small enough for the kernel's 32-bit offsets
                assert 0 <= at[i] < 2 * 64 * D * 2, (S, W, s0, i)


def test_offsets_within_a_page(rows):
    for s0 in (0, 32, 224, 256, 4_000_032):
        k, v, _ = rows(128, s0, 4, 0, 1)
        assert list(zip(k, v)) == [layout(128, s0 % 256 + i) for i in range(32)]
