"""How the reverse walk of an equal-length batch is cut into runs: the plan is host arithmetic (csrc/bwd_plan.hpp) and is
compiled here by the host compiler, no GPU needed.  Every chunk has to be in exactly one run, the sub-runs of the walks
from zero have to cover the chunks after run 0, and no more workgroups are asked for than the chip has places."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_07904_amd", "csrc")
SHIM = """
#include "bwd_plan.hpp"
using namespace hgrn2;
extern "C" int max_runs() { return kMaxLightRuns; }
extern "C" void plan(int BH, int NC, int dk, int dv, int bf16, int places, int* out)
{
    const BwdFusedPlan p = plan_bwd_runs(BH, NC, dk, dv, bf16 != 0, places);
    out[0] = p.R; out[1] = p.rc; out[2] = p.s_sub; out[3] = p.sub_chunks; out[4] = p.seg_tail; out[5] = p.light;
    for (int i = 0; i <= kMaxLightRuns; ++i) out[6 + i] = p.bnd[i];
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("bwd_plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    return ctypes.CDLL(str(d / "shim.so"))


@pytest.mark.parametrize("dk,dv,bf16", [(64, 64, 1), (128, 64, 1), (64, 128, 1), (128, 128, 1), (64, 64, 0)])
def test_runs_cover_every_chunk_and_fit_the_chip(lib, dk, dv, bf16):
    out = (ctypes.c_int * (7 + lib.max_runs()))()
    most = 512 if dk == dv == 64 and bf16 else 256
    for BH in [*range(1, 24), 32, 42, 43, 63, 64, 65, 85, 86, 128, 129, 170, 256, 257, 300, 512, 513, 2000]:
        for NC in [*range(1, 70), 127, 256, 511, 4095, 32768, 70000]:
            for places in (0, 256, 1):
                lib.plan(BH, NC, dk, dv, bf16, places, out)
                R, rc, s_sub, sub, tail, light = out[:6]
                case = (BH, NC, dk, dv, places, list(out))
                assert R >= 1 and (R == 1 or R * BH <= most), case
                assert places != 1 or R == 1, case
                assert places != 256 or R <= max(1, NC // 4), case
                if light:
                    cuts = list(out)[6:7 + R]
                    assert R <= lib.max_runs() and cuts[0] == 0 and cuts[-1] == NC and all(a < b for a, b in zip(cuts, cuts[1:])), case
                else:
                    assert (R - 1) * rc < NC <= R * rc and sub * s_sub == rc, case
                    assert tail == (0 if R == 1 else -(-(NC - rc) // sub)), case
