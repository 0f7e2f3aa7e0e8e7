"""The reverse walk of a training pair cut into runs of one or a few chunks (small batches): light walks by up to 16
runs, and boundaries walked to from zero chunk by chunk; ragged last chunks, every head-dimension pair, both layouts,
gates given and formed in the kernels, in bf16 and fp32, with and without states, 64 and 16 tokens per chunk; with gates
after which nothing of a chunk is left and with gates near one (0.985 to 1: a third after two chunks, 1% after ten), which show
whether a run knows of all chunks after it.  Compared with the fp64 oracle: max|x-y|/max|y| <= 2e-2 per tensor (bf16 storage)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_07904_amd import binding, synth
from gpu_util import TOL, check, dev, host

pytestmark = pytest.mark.gpu
BNHD = binding.HGRN2_LAYOUT_BNHD


@pytest.mark.parametrize("slow", [False, True])
@pytest.mark.parametrize("B,H,N,dk,dv,layout,states,gated,gate,chunk", [
    (1, 2, 65, 128, 128, 0, True, False, "bf16", 0),       # two runs of one chunk, the second of one token
    (2, 3, 640, 128, 128, 1, True, True, "bf16", 0),       # 10 chunks, 10 light runs
    (1, 1, 1009, 128, 128, 0, True, False, "f32", 0),      # 16 chunks from zero, a run each
    (1, 2, 1472, 128, 128, 0, False, True, "bf16", 0),     # 23 chunks from zero, a run each
    (4, 4, 1919, 128, 128, 0, True, True, "bf16", 0),      # 30 chunks, 15 runs of two
    (1, 1, 4097, 128, 64, 0, True, False, "bf16", 0),      # 65 chunks, a run each
    (3, 1, 700, 64, 128, 1, True, False, "bf16", 0),       # 11 chunks
    (1, 2, 1520, 64, 64, 1, True, False, "f32", 0),        # 24 chunks from zero, a run each
    (3, 20, 500, 64, 64, 0, True, True, "bf16", 0),        # 8 chunks, two workgroups on a compute unit
    (2, 2, 150, 64, 64, 1, True, True, "bf16", 16),        # 10 chunks of 16 tokens
])
def test_bwd_saved_in_short_runs(B, H, N, dk, dv, layout, states, gated, gate, chunk, slow):
    print("\n[bwd short runs] B=%d H=%d N=%d dk=%d dv=%d layout=%d chunk=%d slow=%s" % (B, H, N, dk, dv, layout, chunk, slow), flush=True)
    if slow and not gated:
        gate = "f32"                     # (bf16 has four values there)
    w = synth.make_sequence(6100 + N + dk, B, H, N, dk, dv, io_dtype="bf16", gate_dtype=gate, lb=0.985 if slow else 0.3, with_h0=states,
                            with_dO=True, with_dhT=states)
    put = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == BNHD else (lambda t: t)
    get = (lambda t: host(t.permute(0, 2, 1, 3))) if layout == BNHD else host
    rng = np.random.default_rng(6200 + N)
    gates = synth.bf16_round(rng.standard_normal((B, H, N, dk)).astype(np.float32)) if gated else w.f
    beta = rng.uniform(*((0.98, 0.99) if slow else (0.2, 0.9)), size=(H, dk)).astype(np.float32) if gated else None
    q, f, v, dO = put(dev(w.q, "bf16")), put(dev(gates, gate)), put(dev(w.v, "bf16")), put(dev(w.dO, "bf16"))
    h0, dhT = (dev(w.h0), dev(w.dhT)) if states else (None, None)
    bd = torch.from_numpy(beta).cuda() if gated else None
    _, _, saved = binding.hgrn2_fwd_saving(q, f, v, h0, beta=bd, want_hT=False, layout=layout, chunk=chunk)
    dq, df, dv_, dh0, db = binding.hgrn2_bwd_saved(q, f, v, saved, dO, dhT, beta=bd, want_grad_h0=True, layout=layout, chunk=chunk) \
        if gated else (*binding.hgrn2_bwd_saved(q, f, v, saved, dO, dhT, want_grad_h0=True, layout=layout, chunk=chunk), None)
    torch.cuda.synchronize()
    a0, aT = (w.h0, w.dhT) if states else (None, None)
    tol = TOL["bf16"]
    if gated:
        rq, rf, rb, rv, rh = oracle.bwd_gated(w.q, gates, beta, w.v, w.dO, a0, aT)
        check("dbeta", host(db), rb, tol)
    else:
        rq, rf, rv, rh = oracle.bwd(w.q, w.f, w.v, w.dO, a0, aT)
    check("dq", get(dq), rq, tol); check("df", get(df), rf, tol); check("dv", get(dv_), rv, tol)
    check("dh0", host(dh0), rh, tol)
