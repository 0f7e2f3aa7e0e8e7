"""HGRN1 sequences cut into runs (few channels, four blocks of 256 tokens or more): the runs' contributions from zero, chained
into the state every run starts from, forwards and in reverse; lengths around the edges of blocks and runs, both gate types,
with and without states, activations formed inside, and the final state in the place of the initial one (not cut then).
Gates near one, inputs and output gradients with a mean, so that a run still knows of those many runs before (after) it.
Against the fp64 oracle, tolerances as for the uncut walk."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_07904_amd import binding, synth
from gpu_util import TOL, check, dev, host
from test_gpu_hgrn1 import make, make_act, run, run_act

pytestmark = pytest.mark.gpu

SHAPES = [(1, 769, 64), (1, 1024, 320), (2, 1025, 128), (3, 2047, 64), (1, 2100, 1280), (8, 4328, 128), (1, 8192, 64)]


@pytest.mark.parametrize("B,N,d", SHAPES)
def test_hgrn1_in_runs(B, N, d):
    print("\n[hgrn1 runs] B=%d N=%d d=%d" % (B, N, d), flush=True)
    gate = "f32" if N % 2 else "bf16"
    f, i, o, dy, h0, dhN = make(7000 + N, B, N, d, lb=0.9, gate_dtype=gate)
    if d == 320:
        h0 = dhN = None
    run(f, i, o, dy, h0, dhN, gate_dtype=gate)


@pytest.mark.parametrize("B,N,d", SHAPES)
def test_hgrn1_act_in_runs(B, N, d):
    print("\n[hgrn1 act runs] B=%d N=%d d=%d" % (B, N, d), flush=True)
    gate = "bf16" if N % 2 else "f32"
    run_act(*make_act(7100 + N, B, N, d, gate_dtype=gate), gate_dtype=gate)


# Gates of 0.996 to 1: after one run of 256 tokens more than half of a state is left, after eight about 1%, and all of it lies
# around one.  (4 runs, of which the last has one token; 4 of 2 blocks and 5 of 1; 32 and 17 runs, chained eight at a time.)
SLOW = [(1, 769, 64), (2, 2047, 320), (3, 2100, 1280), (1, 8192, 64), (8, 4328, 128)]


def with_mean(x):
    return synth.bf16_round(x + np.float32(1.0))


@pytest.mark.parametrize("B,N,d", SLOW)
def test_hgrn1_in_runs_with_slow_gates(B, N, d):
    print("\n[hgrn1 runs, slow] B=%d N=%d d=%d" % (B, N, d), flush=True)
    f, i, o, dy, h0, dhN = make(7300 + N, B, N, d, lb=0.996, gate_dtype="f32")
    run(f, with_mean(i), o, with_mean(dy), h0, dhN, gate_dtype="f32")


@pytest.mark.parametrize("B,N,d", SLOW)
def test_hgrn1_act_in_runs_with_slow_gates(B, N, d):
    print("\n[hgrn1 act runs, slow] B=%d N=%d d=%d" % (B, N, d), flush=True)
    zf, zi, zo, beta, dy, h0, dhN = make_act(7400 + N, B, N, d)
    beta = np.random.default_rng(7500 + N).uniform(0.994, 0.998, size=d).astype(np.float32)
    run_act(zf, with_mean(zi), zo, beta, with_mean(dy), h0, dhN)


def test_states_continued_in_place():
    f, i, o, dy, h0, dhN = make(7200, 2, 1300, 128, lb=0.996, gate_dtype="f32")
    i, dy = with_mean(i), with_mean(dy)
    fd, idv, od, dyd, s, g = dev(f), dev(i, "bf16"), dev(o, "bf16"), dev(dy, "bf16"), dev(h0), dev(dhN)
    start = s.clone()
    y, hN = binding.hgrn1_fwd(fd, idv, od, s, hN=s)
    gf, gi, go = (torch.empty_like(idv) for _ in range(3))
    need = binding.hgrn1_workspace_bytes(2, 1300, 128)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    p = binding._ptr
    rc = binding.lib().hgrn1_bwd(2, 1300, 128, binding.HGRN2_BF16, binding.HGRN2_F32, p(fd), p(idv), p(od), p(start), p(dyd), p(g),
                                 p(gf), p(gi), p(go), p(g), p(ws), need, binding._stream())
    assert rc == 0
    # and the gradient of the initial state in that state's own place
    other, dhN_d, gf2 = start.clone(), dev(dhN), torch.empty_like(gf)
    rc = binding.lib().hgrn1_bwd(2, 1300, 128, binding.HGRN2_BF16, binding.HGRN2_F32, p(fd), p(idv), p(od), p(other), p(dyd),
                                 p(dhN_d), p(gf2), p(gi), p(go), p(other), p(ws), need, binding._stream())
    assert rc == 0
    torch.cuda.synchronize()
    ry, rh = oracle.hgrn1_fwd(f, i, o, h0)
    rf, ri, ro, rh0 = oracle.hgrn1_bwd(f, i, o, dy, h0, dhN)
    check("y", host(y), ry, TOL["bf16"]); check("hN", host(s), rh, 3e-5)
    check("df", host(gf), rf, TOL["bf16"]); check("dh0", host(g), rh0, 3e-5)
    assert torch.equal(gf, gf2) and torch.equal(g, other)
