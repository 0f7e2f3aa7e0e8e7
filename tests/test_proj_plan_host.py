"""Which tile a product of the projections takes and into how many shares dW3's contraction over the tokens is cut: the plan is
host arithmetic (csrc/proj_plan.hpp) and is compiled here by the host compiler, no GPU needed.  Every share has to have steps,
tiles have to divide the result, the shares' room stays bounded, and the shapes of the GPU tests take the plans they are there for."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_07904_amd", "csrc")
SHIM = """
#include "proj_plan.hpp"
using namespace hgrn2;
extern "C" void plan(int M, int N, int K, int may_split, int* out) { const NtPlan p = plan_nt(M, N, K, may_split != 0); out[0] = p.tile; out[1] = p.splits; }
extern "C" int rows(int M, int d) { return act_rows(M, d); }
"""
WIDTHS = range(256, 4097, 256)
TOKENS = [*range(1, 70), 127, 128, 129, 500, 1000, 1500, 2047, 2048, 3456, 4097, 8192, 14720, 16384, 40000, 1 << 20, 1 << 22]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("proj_plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    return ctypes.CDLL(str(d / "shim.so"))


def plan(lib, M, N, K, may_split):
    out = (ctypes.c_int * 2)()
    lib.plan(M, N, K, int(may_split), out)
    return out[0], out[1]


def padded(M):
    return (M + 63) // 64 * 64


def test_tiles_divide_and_every_share_has_steps(lib):
    for d in WIDTHS:
        for M in TOKENS:
            for product, (m, n, k, split) in {"projection": (M, 3 * d, d, False), "dx": (M, d, 3 * d, False),
                                              "dw": (3 * d, d, padded(M), True)}.items():
                tile, shares = plan(lib, m, n, k, split)
                case = (product, M, d, tile, shares)
                assert tile in (64, 128, 256) and n % tile == 0 and k % 64 == 0, case
                assert shares == 1 or (split and shares in (2, 4, 8, 16)), case
                steps = k // 64
                cuts = [s * steps // shares for s in range(shares + 1)]
                assert cuts[0] == 0 and cuts[-1] == steps and all(b > a for a, b in zip(cuts, cuts[1:])), case
                assert shares == 1 or 4 * m * n * shares <= 64e6, case
                # rows of dW3's tiles: 192 (wide), 128 or 64; none is ragged there
                assert not split or m % (192 if tile == 256 else tile) == 0, case
            assert lib.rows(M, d) in (32, 64) and padded(M) % lib.rows(M, d) == 0


# (tokens, width): (projection's tile, dx's tile, dW3's tile and shares), as tests/test_gpu_proj.py relies on them
GPU_SHAPES = {
    (1, 256): (64, 64, 64, 1), (1500, 512): (128, 64, 64, 1), (4100, 256): (128, 64, 64, 4), (2048, 1024): (128, 64, 128, 1),
    (4097, 1280): (256, 128, 256, 1), (9000, 1024): (256, 256, 128, 1), (3500, 768): (128, 128, 128, 2), (4900, 512): (128, 128, 128, 4),
    (9984, 256): (128, 128, 128, 16), (5633, 1280): (128, 128, 256, 2), (14720, 1024): (256, 256, 256, 4),
}


@pytest.mark.parametrize("shape", GPU_SHAPES)
def test_plans_of_the_gpu_tests(lib, shape):
    M, d = shape
    got = (plan(lib, M, 3 * d, d, False)[0], plan(lib, M, d, 3 * d, False)[0], *plan(lib, 3 * d, d, padded(M), True))
    assert got == GPU_SHAPES[shape]
    steps, shares = padded(M) // 64, got[3]
    assert shares == 1 or steps % shares != 0          # shares of unequal length
