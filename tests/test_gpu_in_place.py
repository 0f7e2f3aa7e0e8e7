"""A state continued in place: hT is h0's buffer (forward), grad_h0 is grad_hT's (backward).  The workgroups that
share a sequence must not start from a state another one of them has replaced, so such calls are cut another
way; sizes are those at which the usual cut shares a sequence: runs with light walks, runs from walks from zero
(few and many), the fp32 read-out from contributions, spans of a packed batch, two runs of 64-wide heads.
Against the oracle, bounds of gpu_util; the kept states are checked through the gradients."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_07904_amd import binding, synth
from gpu_util import TOL, check, dev, host

pytestmark = pytest.mark.gpu

# (B, H, N, dk, dv, storage)
CASES = [
    (1, 3, 777, 128, 128, "bf16"),       # light walks, halves of dv
    (5, 13, 460, 128, 128, "bf16"),      # light walks, whole dv
    (1, 100, 330, 64, 64, "bf16"),       # two light runs
    (1, 3, 3001, 128, 128, "bf16"),      # walks from zero, added up by the runs
    (1, 1, 4481, 64, 128, "bf16"),       # walks from zero, with the carry kernel
    (1, 1, 64, 128, 64, "bf16"),         # one chunk
    (2, 3, 300, 64, 64, "f32"),          # read-out from contributions
    (1, 2, 2100, 64, 64, "f32"),         # fp32 runs
]


@pytest.mark.parametrize("B,H,N,dk,dv,io", CASES)
def test_forward_state_in_place(B, H, N, dk, dv, io):
    print("\n[in place] B=%d H=%d N=%d dk=%d dv=%d %s" % (B, H, N, dk, dv, io), flush=True)
    w = synth.make_sequence(5000 + N, B, H, N, dk, dv, io_dtype=io, lb=0.9, with_h0=True, with_dO=True)
    q, f, v = dev(w.q, io), dev(w.f, io if io == "f32" else "bf16"), dev(w.v, io)
    ro, rhT = oracle.fwd(w.q, w.f, w.v, w.h0)
    saving = io == "bf16" or dk == dv == 64
    for saved in ([False, True] if saving else [False]):
        state = dev(w.h0)
        if saved:
            o, hT, kept = binding.hgrn2_fwd_saving(q, f, v, state, hT=state)
        else:
            o, hT = binding.hgrn2_fwd(q, f, v, state, hT=state)
        torch.cuda.synchronize()
        assert hT is state
        check("o", host(o), ro, TOL[io])
        check("hT", host(state), rhT, TOL[io])
    if saving:
        g = binding.hgrn2_bwd_saved(q, f, v, kept, dev(w.dO, io))
        torch.cuda.synchronize()
        for name, x, r in zip(("dq", "df", "dv"), g, oracle.bwd(w.q, w.f, w.v, w.dO, w.h0, None)):
            check(name, host(x), r, TOL[io])


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 128)])
@pytest.mark.parametrize("lens", [[5, 700, 64, 0, 1], [0, 900, 200]])
def test_packed_forward_state_in_place(lens, dk, dv):
    print("\n[in place, packed] lens=%s dk=%d dv=%d" % (lens, dk, dv), flush=True)
    H, T, B = 64, sum(lens), len(lens)
    w = synth.make_sequence(5100 + T, 1, H, T, dk, dv, io_dtype="bf16", lb=0.9, with_dO=True)
    h0 = (0.1 * np.random.default_rng(T).standard_normal((B, H, dk, dv))).astype(np.float32)
    q, f, v, dO = (dev(x, "bf16")[0].permute(1, 0, 2).contiguous() for x in (w.q, w.f, w.v, w.dO))
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), device="cuda")
    saved = torch.full((binding.hgrn2_saved_states_varlen_bytes(binding.make_shape_varlen(q, v, f, B)),), 0xFF,
                       dtype=torch.uint8, device="cuda")
    s1, s2 = dev(h0), dev(h0)
    o, _ = binding.hgrn2_fwd_varlen(q, f, v, cu, s1, hT=s1)
    o2, _ = binding.hgrn2_fwd_varlen(q, f, v, cu, s2, hT=s2, saved_states=saved)
    g = binding.hgrn2_bwd_varlen(q, f, v, dO, cu, dev(h0), saved_states=saved)
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and torch.equal(s1, s2)
    at = 0
    for b, n in enumerate(lens):
        s = slice(at, at + n)
        at += n
        if n == 0:
            assert np.array_equal(host(s1[b]), h0[b].astype(np.float64))
            continue
        cut = lambda x: x[:, :, s]
        ro, rhT = oracle.fwd(cut(w.q), cut(w.f), cut(w.v), h0[b:b + 1])
        check("o[%d]" % b, host(o[s].permute(1, 0, 2)[None]), ro, TOL["bf16"])
        check("hT[%d]" % b, host(s1[b:b + 1]), rhT, TOL["bf16"])
        for name, x, r in zip(("dq", "df", "dv"), g, oracle.bwd(cut(w.q), cut(w.f), cut(w.v), cut(w.dO), h0[b:b + 1], None)):
            check("%s[%d]" % (name, b), host(x[s].permute(1, 0, 2)[None]), r, TOL["bf16"])


# 130 heads of 64 (usually three runs), 33 of 128 (seven), one long one (28 runs); with kept states and without,
# and with the reduction of the gradient of beta that the number of runs enters
@pytest.mark.parametrize("B,H,N,dk,gated", [(2, 65, 800, 64, False), (2, 65, 800, 64, True), (1, 33, 2000, 128, False), (1, 1, 7200, 128, True)])
def test_backward_state_gradient_in_place(B, H, N, dk, gated):
    print("\n[in place, backward] B=%d H=%d N=%d d=%d gated=%d" % (B, H, N, dk, gated), flush=True)
    w = synth.make_sequence(5200 + N, B, H, N, dk, dk, io_dtype="bf16", lb=0.9, with_h0=True, with_dO=True)
    q, f, v, dO = (dev(x, "bf16") for x in (w.q, w.f, w.v, w.dO))
    beta = None
    if gated:
        f = dev(np.random.default_rng(N).standard_normal(w.f.shape), "bf16")          # pre-activations
        beta = torch.full((H, dk), 0.9, device="cuda")
    h0 = dev(w.h0)
    dhT = 0.1 * torch.randn(B, H, dk, dk, device="cuda", generator=torch.Generator(device="cuda").manual_seed(N))
    kept = binding.hgrn2_fwd_saving(q, f, v, h0, beta=beta)[2]
    apart = binding.hgrn2_bwd_saved(q, f, v, kept, dO, dhT, beta=beta, want_grad_h0=True)
    g1, g2 = dhT.clone(), dhT.clone()
    a = binding.hgrn2_bwd_saved(q, f, v, kept, dO, g1, beta=beta, grad_h0=g1)
    if gated:
        x = binding.hgrn2_bwd_gated(q, f, beta, v, dO, h0, g2, grad_h0=g2)
        b = (x[0], x[1], x[3], x[4], x[2])
    else:
        b = binding.hgrn2_bwd(q, f, v, dO, h0, g2, grad_h0=g2)
    torch.cuda.synchronize()
    assert a[3] is g1 and b[3] is g2
    # two correct cuts differ by the rounding of the states at the run boundaries: the bound of one of them, twice
    for name, r, x, y in zip(("dq", "df", "dv", "dh0", "dbeta"), apart, a, b):
        check(name, host(x), host(r), 2 * TOL["bf16"])
        check(name + " stateless", host(y), host(r), 2 * TOL["bf16"])
    if not gated:
        for name, x, r in zip(("dq", "df", "dv", "dh0"), a, oracle.bwd(w.q, w.f, w.v, w.dO, w.h0, host(dhT).astype(np.float32))):
            check(name, host(x), r, TOL["bf16"])
