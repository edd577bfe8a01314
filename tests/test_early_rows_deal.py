"""Host-side check (no GPU needed) of how the channels of a launch with early rows are dealt to its
splits: every channel to exactly one split, waves ascending, and no split with much more than its
share of what is kept where the kept channels lie together or repeat with the heads.  (A split that
owns one contiguous range has up to S times its share then.)  The index arithmetic is the kernels'
own, compiled for the host."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2504_08378_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
SOURCE = """
#include <hip/hip_runtime.h>
#include "af_internal.h"
extern "C" int wave_channels(int n, int S, int s, int w, int waves, int* out, int* first, int* end) {
  const int cycles = af_dealt_cycles(n, S), q0 = af_dealt_cycle(cycles, w, waves), q1 = af_dealt_cycle(cycles, w + 1, waves);
  for (int l = 0; l < (q1 - q0) * AF_DEAL; ++l) out[l] = af_dealt_channel(q0, S, s, w, l);
  *first = q0 * S * AF_DEAL;
  *end = q1 * S * AF_DEAL;
  return (q1 - q0) * AF_DEAL;
}
"""
WAVES = 16


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("deal")
    src, so = str(d / "deal.hip"), str(d / "deal.so")
    open(src, "w").write(SOURCE)
    subprocess.run([HIPCC, *build.HIPCC_FLAGS, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-shared", src,
                    "-o", so], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    return ctypes.CDLL(so)


def _owners(lib, n, S):
    """split of every channel; checks that the channels of a wave ascend and that all are dealt once"""
    owner = np.full(n, -1)
    for s in range(S):
        before, stretch_end = -1, 0
        for w in range(WAVES):
            ch, first, end = np.zeros(n + 64, np.int32), ctypes.c_int(), ctypes.c_int()
            own = lib.wave_channels(n, S, s, w, WAVES, ch.ctypes.data_as(ctypes.c_void_p), ctypes.byref(first), ctypes.byref(end))
            assert first.value == stretch_end
            stretch_end = end.value
            ch = ch[:own]
            assert np.all(np.diff(np.concatenate([[before], ch])) > 0)
            before = ch[-1] if own else before
            assert np.all((ch >= first.value) & (ch < end.value))
            ch = ch[ch < n]
            assert np.all(owner[ch] == -1)
            owner[ch] = s
        assert stretch_end >= n
    assert np.all(owner >= 0)
    return owner


@pytest.mark.parametrize("n", [8, 64, 136, 1000, 2048, 4088, 4096, 4104, 11008, 16392, 28672, 32768])
@pytest.mark.parametrize("S", [1, 2, 3, 5, 8, 16, 61, 256])
def test_every_channel_is_dealt_once(lib, n, S):
    _owners(lib, n, S)


@pytest.mark.parametrize("n,S", [(4096, 3), (4096, 4), (4096, 6), (5120, 4), (8192, 4), (8192, 6), (11008, 6), (11008, 8),
                                 (13824, 6), (14336, 8), (28672, 4), (28672, 8)])
def test_kept_channels_that_lie_together_are_spread(lib, n, S):
    owner, i = _owners(lib, n, S), np.arange(n)
    kept = {"first half": i < n // 2, "last fifth": i > 0.8 * n}
    for hd in (64, 128):
        m = i % hd
        kept[f"half of the heads of {hd}"] = (np.random.default_rng(n).random(n // hd + 1) < 0.5)[i // hd]
        kept[f"half of every head of {hd}"] = m < hd // 2
        kept[f"a quarter of every head of {hd}"] = (m >= hd // 4) & (m < hd // 2)
    for p in (16, 32, 64, 256, 512, 1024):
        kept[f"every other block of {p}"] = (i // p) % 2 == 0
    for what, k in kept.items():
        c = np.bincount(owner[k], minlength=S)
        assert c.max() <= 1.35 * c.mean(), (what, c)
