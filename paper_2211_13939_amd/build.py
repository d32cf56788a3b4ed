"""Build the C-ABI library (HIP kernels + host code) for gfx950 into
paper_2211_13939_amd/libtts_pool.so.  Run on the CPU machine; hipcc cross-compiles."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libtts_pool.so")
SOURCES = ["kernels.hip", "segment.hip", "segment32.hip", "tts_pool.cpp", "postnet.hip", "postnet.cpp", "vocoder.hip", "vocoder.cpp", "encoder.hip", "encoder.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # the first 16 dwords of a kernel's arguments arrive in scalar registers with the wave (gfx950 preloads them):
         # the first loads of a kernel no longer wait for a cold read of the argument block
         "-mllvm", "-amdgpu-kernarg-preload-count=16",
         # accumulators of the matrix instructions in ordinary vector registers.  Left to its heuristics the compiler keeps them in the
         # accumulation half of the file in the vocoder's up-samplings and its last layer, with 544 moves in and out (none with the
         # option): a two-byte call of 128 windows of 48 frames 512 -> 509 us, of 256 1049 -> 1040; up to 64 windows, in fp32 and in the
         # other files, whose kernels hold no such moves either way, the times are the same
         "-mllvm", "-amdgpu-mfma-vgpr-form=1",
         "-Wall", "-Wno-unused-result"]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def build(verbose: bool = False) -> str:
    cmd = [HIPCC] + FLAGS + ["-x", "hip"] + sources() + ["-o", OUT]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
