"""How the forward walk of an equal-length batch is cut into runs, for every chunk count the library accepts:
the plan is host arithmetic (csrc/fwd_plan.hpp) and is compiled here by the host compiler, no GPU needed.
Runs with light walks have to rise from 0 to the number of chunks; runs of equal length have to cover it."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_07904_amd", "csrc")
SHIM = """
#include "fwd_plan.hpp"
using namespace hgrn2;
extern "C" int max_runs() { return kMaxFwdRuns; }
// out: light, seg, run_chunks, then the light runs' cuts
extern "C" void plan(int BH, int NC, int dk, int dv, int light_walks, int kept, int* out)
{
    const FwdRuns r = plan_fwd_runs(BH, NC, dk, dv, light_walks != 0, kept != 0);
    out[0] = r.light; out[1] = r.seg; out[2] = r.run_chunks;
    FwdCuts c = {};
    if (r.light > 1) fused_cuts(NC, r.light, &c);
    for (int i = 0; i <= kMaxFwdRuns; ++i) out[3 + i] = c.bnd[i];
}
extern "C" int grid_of(int BH, int per) { return run_grid(BH, per); }
extern "C" int item_of(int block, int BH, int per) { const RunItem r = run_item(block, BH, per); return r.seq * per + r.sub; }
"""
INT_MAX = 2 ** 31 - 1


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("fwd_plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    return ctypes.CDLL(str(d / "shim.so"))


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 64), (64, 128), (128, 128)])
def test_cuts_rise_and_cover_every_chunk(lib, dk, dv):
    runs = lib.max_runs()
    out = (ctypes.c_int * (4 + runs))()
    for BH in [*range(1, 24), 32, 42, 43, 50, 63, 64, 65, 85, 86, 96, 127, 128, 129, 256, 300, 2000]:
        most = min(INT_MAX // 2 // BH, (INT_MAX // 8 + 7) // 8)          # what the shape check accepts: chunks of 8 tokens
        for NC in [*range(1, 70), 127, 256, 511, 4095, 32766, 32767, 32768, 40000, 65535, 65536, 65540, 70000, 1 << 20, most - 1, most]:
            if NC > most:
                continue
            lib.plan(BH, NC, dk, dv, 1, 0, out)
            light, seg, run_chunks, bnd = out[0], out[1], out[2], list(out)[3:]
            case = (BH, NC, dk, dv, light, seg, run_chunks, bnd)
            assert 1 <= light <= runs and 1 <= seg <= max(1, NC) and (light == 1 or seg == 1), case
            if light > 1:
                cuts = bnd[:light + 1]
                assert cuts[0] == 0 and cuts[-1] == NC and all(a < b for a, b in zip(cuts, cuts[1:])), case
            if seg > 1:
                assert (seg - 1) * run_chunks < NC <= seg * run_chunks, case
            # a state continued in place: no light walks, and the runs' states (fp32, with their gate products)
            # fit the room of the chunk states (bf16)
            lib.plan(BH, NC, dk, dv, 0, 0, out)
            light, seg, run_chunks = out[0], out[1], out[2]
            case = (BH, NC, dk, dv, light, seg, run_chunks)
            assert light == 1 and seg >= 1 and (seg - 1) * run_chunks < NC <= seg * run_chunks, case
            assert seg == 1 or seg * (4 * dk * dv + 4 * dk) <= NC * 2 * dk * dv, case


def test_light_runs_are_dealt_evenly_to_the_xcds(lib):
    """Every (sequence, run, half) is somebody's, and the workgroups of an XCD (every eighth one) are an eighth of all:
    32 at most, one per compute unit, for the 256 a plan fills."""
    for BH in [*range(1, 130), 1000]:
        for per in range(1, 33):
            items, grid = BH * per, lib.grid_of(BH, per)
            if items > 1100:
                continue
            got = [lib.item_of(b, BH, per) for b in range(grid)]
            assert items <= grid < items + 8 and sorted(got) == list(range(grid)), (BH, per)
            for x in range(8):
                assert sum(i < items for i in got[x::8]) <= (items + 7) // 8, (BH, per, x)
    out = (ctypes.c_int * (4 + lib.max_runs()))()
    for dk, dv in ((64, 64), (128, 64), (64, 128), (128, 128)):
        for BH in range(1, 257):
            for NC in (8, 16, 32, 64, 300):
                lib.plan(BH, NC, dk, dv, 1, 0, out)
                assert out[0] == 1 or out[0] * BH <= 256, (BH, NC, dk, dv, out[0])


def test_kept_states_never_change_what_the_workspace_is_sized_for(lib):
    """The workspace depends on the shape alone: a walk that keeps states is cut into the same runs of equal length, or
    not at all."""
    a, b = ((ctypes.c_int * (4 + lib.max_runs()))() for _ in range(2))
    for dk, dv in ((64, 64), (128, 64), (64, 128), (128, 128)):
        for BH in range(1, 140):
            for NC in (2, 13, 32, 55, 56, 64, 300, 4000):
                for light in (0, 1):
                    lib.plan(BH, NC, dk, dv, light, 0, a)
                    lib.plan(BH, NC, dk, dv, light, 1, b)
                    assert list(a) == list(b) or (b[0] == 1 and b[1] == 1), (BH, NC, dk, dv, light)
                    assert list(a) == list(b) or (dk == dv == 128 and BH > 112 and NC >= 56), (BH, NC, dk, dv, light)
