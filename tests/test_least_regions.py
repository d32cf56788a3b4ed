"""Workgroups of a launch of the vocoder's smallest regions (csrc/vocoder_kernels.h): one for every region of every block and window, a block's dealt
evenly over the eight XCDs.  Host arithmetic only."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "vocoder_kernels.h"
extern "C" int all(int windows, int positions) { return tts::voc_least(windows, positions).all(); }
extern "C" int block(int windows, int positions, int i, int* window, int* tile) { return tts::voc_least(windows, positions).block(i, window, tile); }
"""
OUT = (104, 56, 8)              # positions of a region of 128 that two halos of 12, 36 and 60 leave


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("regions")
    src = d / "regions.cpp"
    src.write_text(SOURCE)
    out = str(d / "libregions.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2211_13939_amd", "csrc"), "-Wno-unused-result", str(src), "-o", out], check=True)
    return C.CDLL(out)


@pytest.mark.parametrize("windows,frames", [(1, 1), (1, 100), (2, 7), (3, 48), (6, 24), (20, 16), (40, 8), (7, 13), (45, 1), (256, 1)])
def test_every_region_has_one_workgroup(lib, windows, frames):
    positions = 8 * frames
    want = {(b, w, t) for b in range(3) for w in range(windows) for t in range(-(-positions // OUT[b]))}
    n = lib.all(windows, positions)
    got, xcd = [], {b: np.zeros(8, int) for b in range(3)}
    for i in range(n):
        w, t = C.c_int(), C.c_int()
        b = lib.block(windows, positions, i, C.byref(w), C.byref(t))
        got.append((b, w.value, t.value))
        xcd[b][i % 8] += 1
    assert len(got) == len(want) and set(got) == want
    assert [b for b, _, _ in got] == sorted((b for b, _, _ in got), reverse=True)       # the longest kernel's first
    assert all(x.max() - x.min() <= 1 for x in xcd.values())
