"""How HGRN1's sequences are cut into runs of whole blocks: host arithmetic (csrc/hgrn1_plan.hpp), compiled here by the host
compiler, no GPU needed.  Every block has to be in exactly one run, no run may be empty, and no more workgroups are asked for
than the chip has places."""
import ctypes
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_07904_amd", "csrc")
SHIM = """
#include "hgrn1_plan.hpp"
using namespace hgrn2;
extern "C" int runs(int B, int d, int blocks, int* per) { return h1_runs(B, d, blocks, per); }
extern "C" int blocks(int N, int longer) { return h1_blocks(N, longer ? kH1SegLong : kH1SegShort); }
"""


def test_runs_cover_every_block(tmp_path):
    (tmp_path / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(tmp_path / "shim.cpp"), "-o", str(tmp_path / "shim.so")])
    lib = ctypes.CDLL(str(tmp_path / "shim.so"))
    per = ctypes.c_int()
    cut = 0
    for d in (64, 128, 192, 320, 1024, 2048, 5440, 5504, 1 << 20):
        for B in (1, 2, 3, 5, 8, 28, 42, 43, 85, 86, 128, 256, 257, 1000):
            for N in [*range(1, 1400, 97), 768, 769, 1024, 1025, 2048, 4328, 8192, 16384, 16385, 100000, 1 << 24]:
                for longer in (0, 1):
                    NB = lib.blocks(N, longer)
                    block = 512 if longer else 256
                    assert (NB - 1) * block < N <= NB * block
                    R = lib.runs(B, d, NB, ctypes.byref(per))
                    case = (B, N, d, NB, R, per.value)
                    assert R >= 1 and (R - 1) * per.value < NB <= R * per.value, case
                    if R > 1:
                        cut += 1
                        assert R <= 64 and R * B * (d // 64) <= 256 and NB >= 4, case
                        # the walk from zero takes 256 tokens a block whatever the walk proper takes: its last run has tokens
                        assert (R - 1) * per.value * block < N, case
    assert cut > 100
