"""Where the reverse walk finds the rows of a chunk (csrc/walk_rows.hpp, compiled here by the host compiler, no GPU needed):
32-bit byte offsets inside a descriptor that covers exactly the chunk's tokens.  At every stride the walk takes them for, up to the
last one, a row that stands for a token lies where 64-bit arithmetic says, and all of a row that stands for none lies outside
the descriptor; beyond it the walk is told that they do not reach, and such a batch is not cut into runs."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_07904_amd", "csrc")
SHIM = """
#include "bwd_plan.hpp"
#include "walk_rows.hpp"
using namespace hgrn2;
extern "C" int near_rows(long long ld_k, long long ld_v, int gate_bytes) { return walk_rows_near(ld_k, ld_v, gate_bytes); }
extern "C" int runs(int BH, int NC, int dk, int dv) { return plan_bwd_runs(BH, NC, dk, dv, true, 0).R; }
// -1: all rows lie right; else the first row that does not
extern "C" int wrong_row(int lo, int hi, int ld, int width, int es)
{
    const uint32_t bytes = walk_chunk_bytes(hi - lo, ld, width, es);
    if (bytes != ((unsigned long long)(hi - lo - 1) * ld + width) * es) return 1000;
    for (int row = 0; row < kWalkRows; ++row)
        for (int col = 0; col < width; col += width - 1) {
            const uint32_t at = walk_row_offset(row, lo, ld, col, es);
            const bool token = row >= lo && row < hi;
            const long long true_at = ((long long)(row - lo) * ld + col) * es;
            if (token ? (long long)at != true_at || at + (unsigned)es > bytes : at < bytes) return row;
        }
    return -1;
}
"""
LAST = 2 ** 31 // 8          # strides beyond this one are refused (in elements)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk_rows")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-fsanitize=signed-integer-overflow", "-fno-sanitize-recover",
                           "-static-libubsan", "-I" + CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    so = ctypes.CDLL(str(d / "shim.so"))
    so.near_rows.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    return so


@pytest.mark.parametrize("width", [64, 128])
@pytest.mark.parametrize("es", [2, 4])
def test_rows_of_every_stride_lie_right_or_are_not_taken(lib, width, es):
    last = max(h for h in range(1, LAST // width + 1) if lib.near_rows(h * width, 0, es)) * width if es == 4 else 0
    if es == 2:
        h = 1
        while lib.near_rows(2 * h * width, 0, 2):
            h *= 2
        last = next(x for x in range(2 * h - 1, h - 1, -1) if lib.near_rows(x * width, 0, 2)) * width
    assert 64 * last * es < 2 ** 31 <= 64 * (last + width) * es
    strides = sorted({width, 2 * width, 16 * width, 1000 * width, last // 2 // width * width, last - width, last})
    for ld in strides:
        for lo, hi in [(0, 64), (0, 1), (0, 63), (24, 40), (24, 25), (16, 48), (28, 36), (63, 64)]:
            assert lib.wrong_row(lo, hi, ld, width, es) == -1, (lo, hi, ld)


def test_far_rows_are_told_apart(lib):
    assert lib.near_rows(64, 64, 2) and lib.near_rows(65535 * 128, 65535 * 128, 4) and lib.near_rows(131071 * 128, 64, 2)
    assert not lib.near_rows(65536 * 128, 64, 4) and not lib.near_rows(131072 * 128, 64, 2)
    assert not lib.near_rows(64, 131072 * 128, 2)                 # (wide values beside narrow keys)
    assert not lib.near_rows(LAST, LAST, 2) and not lib.near_rows(LAST, LAST, 4)


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 64), (64, 128), (128, 128)])
def test_so_many_heads_are_one_run_each(lib, dk, dv):
    heads = next(h for h in range(1, LAST // 64) if not lib.near_rows(h * dk, h * dv, 4))
    assert heads > 512
    for BH in (heads, 2 * heads, LAST // max(dk, dv)):
        for NC in (1, 2, 7, 100):
            assert lib.runs(BH, NC, dk, dv) == 1
