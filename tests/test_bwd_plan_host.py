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
extern "C" void plan(int BH, int NC, int dk, int dv, int bf16, int places, int fine, int* out)
{
    const BwdFusedPlan p = plan_bwd_runs(BH, NC, dk, dv, bf16 != 0, places, fine != 0);
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
            for places, fine in ((0, 0), (0, 1), (256, 0), (1, 0)):
                lib.plan(BH, NC, dk, dv, bf16, places, fine, out)
                R, rc, s_sub, sub, tail, light = out[:6]
                case = (BH, NC, dk, dv, places, fine, list(out))
                if fine:          # needs no other room than the plan of 64 tokens per chunk: the same plan, or light
                    usual = (ctypes.c_int * len(out))()
                    lib.plan(BH, NC, dk, dv, bf16, places, 0, usual)
                    assert list(out) == list(usual) or out[0] == 1 or out[5], (case, list(usual))
                assert R >= 1 and (R == 1 or R * BH <= most), case
                assert places != 1 or R == 1, case
                assert places != 256 or R <= max(1, NC // 4), case
                if light:
                    cuts = list(out)[6:7 + R]
                    assert R <= lib.max_runs() and cuts[0] == 0 and cuts[-1] == NC and all(a < b for a, b in zip(cuts, cuts[1:])), case
                else:
                    assert (R - 1) * rc < NC <= R * rc and sub * s_sub == rc, case
                    assert tail == (0 if R == 1 else -(-(NC - rc) // sub)), case


# us of the reverse walk of a training pair at some sizes, cut into light runs (L) or runs from zero (E), as measured on an MI355X
# (one run to the next: 1%) with the walk that the plan's costs are fitted to, the one before the present walk of bf16 storage
MEASURED = [
    (64, 64, 1, 256, {"E64": 46.7, "E128": 46.5, "E256": 63.0}),
    (128, 128, 1, 256, {"E64": 67.0, "E128": 61.0, "E256": 76.8}),
    (128, 64, 1, 256, {"E64": 55.6, "E128": 52.3, "E256": 68.4}),
    (64, 128, 1, 256, {"E64": 61.9, "E128": 55.1, "E256": 70.3}),
    (64, 64, 128, 12, {"L2": 40.0, "L3": 37.8, "L4": 38.6}),
    (64, 64, 80, 20, {"L3": 50.6, "E5": 48.4, "L5": 45.9, "L6": 46.2}),
    (64, 64, 120, 20, {"L4": 55.7, "E4": 57.4}),
    (64, 128, 48, 32, {"L5": 87.6, "E5": 81.7}),
    (64, 128, 1, 12, {"L12": 32.5, "E12": 25.4, "L6": 34.0, "E6": 33.1}),
    (128, 64, 48, 32, {"L5": 71.1, "E5": 72.1}),
    (128, 128, 56, 40, {"L4": 118.4, "E4": 122.5}),
]


@pytest.mark.parametrize("dk,dv,BH,NC,us", MEASURED)
def test_the_cut_is_one_of_the_fast_ones(lib, dk, dv, BH, NC, us):
    out = (ctypes.c_int * (7 + lib.max_runs()))()
    lib.plan(BH, NC, dk, dv, 1, 0, 0, out)
    cut = "%s%d" % ("L" if out[5] else "E", out[0])
    assert cut in us and us[cut] <= 1.03 * min(us.values()), (cut, us)


def test_a_fine_length_is_one_launch_where_few_runs_have_four_chunks(lib):
    out = (ctypes.c_int * (7 + lib.max_runs()))()
    for dk, dv in ((64, 64), (128, 128)):
        places = 512 if dk == 64 else 256
        for BH in range(1, 260):
            for NC in (1, 2, 8, 12, 16, 24, 48, 64, 100):
                lib.plan(BH, NC, dk, dv, 1, 0, 1, out)
                runs, light = out[0], out[5]
                if min(places // BH, NC // 4) <= 4:
                    assert runs == 1 or light, (dk, BH, NC, list(out))
