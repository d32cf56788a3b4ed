"""The words of a small call's one launch (csrc/conv5_chain.h): a PostNet or an encoder has room for those of every call it accepts.
Host arithmetic only, compiled from the header that sizes the arena and chooses a call's column groups."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "postnet_kernels.h"
extern "C" size_t set_bytes(int value_bytes, long columns, int layers) { return tts::chain_set_bytes(value_bytes, columns, layers); }
extern "C" size_t call_bytes(int value_bytes, int columns, int layers) { return tts::chain_call_bytes(value_bytes, columns, layers); }
extern "C" int most_columns(int value_bytes) { return tts::chain_most_columns(value_bytes); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("words")
    src = d / "words.cpp"
    src.write_text(SOURCE)
    out = str(d / "libwords.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2211_13939_amd", "csrc"), "-Wno-unused-result", str(src), "-o", out], check=True)
    L = C.CDLL(out)
    for f in (L.set_bytes, L.call_bytes):
        f.restype = C.c_size_t
    L.set_bytes.argtypes = [C.c_int, C.c_long, C.c_int]
    L.call_bytes.argtypes = [C.c_int, C.c_int, C.c_int]
    return L


def _stored(value_bytes, columns, layers):
    """Every column group of a call stores all of its columns, padding included: 512 channels a layer.  A group is one, two or three times
    two column tiles of 16 (fp32: one), the fewest that leave eight groups at most."""
    unit = 2 if value_bytes == 2 else 1
    for times in (1, 2, 3):
        cols = 16 * unit * times
        groups = -(-columns // cols)
        if groups <= 8:
            return groups * cols * layers * 512 * value_bytes
    raise AssertionError("no such call")


@pytest.mark.parametrize("layers", [3, 4])                 # the encoder's and the PostNet's
@pytest.mark.parametrize("value_bytes", [2, 4])
def test_every_call_fits_the_words_of_its_object(lib, value_bytes, layers):
    most = lib.most_columns(value_bytes)
    assert most == (768 if value_bytes == 2 else 384)
    need = 0
    for columns in range(1, 1025):                         # an object made for this many columns, and every call it accepts
        if columns <= most:
            assert lib.call_bytes(value_bytes, columns, layers) == _stored(value_bytes, columns, layers)
            need = max(need, _stored(value_bytes, columns, layers))
        assert lib.set_bytes(value_bytes, columns, layers) >= need, columns
