"""How the forward walk of bf16 batches is cut: runs with a light walk of their own, runs whose entering
states come from walks from zero (added up by the runs' workgroups, or by the carry kernel when there
are many), spans of a packed batch that start and end inside sequences; heads of 64 (workgroups of four
waves).  Against the oracle, at the sizes where a cut can go wrong: one chunk per run, ragged last
chunks, fewer chunks than runs, an initial and a final state.  Tolerance: the bf16 bound of gpu_util.
The states kept for the backward pass are checked through its gradients."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_07904_amd import binding, synth
from gpu_util import TOL, check, dev, host

pytestmark = pytest.mark.gpu


# (B, H, N, dk, dv, gate dtype): what the cut is for it
CASES = [
    (1, 1, 65, 64, 64, "bf16"),          # two chunks, two light runs of one chunk
    (1, 3, 777, 128, 128, "bf16"),       # 13 chunks, ragged: light runs, halves of dv
    (2, 20, 460, 128, 128, "f32"),       # three light runs of each of 40 sequences, halves of dv
    (5, 13, 460, 128, 128, "f32"),       # the same of 65 sequences, whole dv
    (1, 2, 1000, 64, 64, "f32"),         # 16 chunks of 64-wide heads
    (1, 2, 700, 128, 64, "bf16"),
    (1, 2, 700, 64, 128, "f32"),
    (1, 2, 2100, 64, 64, "bf16"),        # 33 chunks: walks from zero in eleven runs of three
    (1, 6, 2700, 64, 64, "bf16"),        # 43 chunks in eleven runs of four, the last one of three
    (1, 3, 3001, 128, 128, "bf16"),      # 47 chunks in twelve runs, the last one shorter
    (1, 64, 4100, 128, 128, "bf16"),     # 65 chunks in four runs, whole dv
    (1, 1, 4481, 64, 128, "bf16"),       # 71 chunks: 17 runs and more, with the carry kernel
    (5, 17, 460, 128, 128, "bf16"),      # 85 sequences in three light runs: no whole number of sequences to an XCD
    (1, 25, 700, 64, 128, "bf16"),       # the same in halves of dv
    (3, 29, 300, 64, 64, "f32"),
]


@pytest.mark.parametrize("B,H,N,dk,dv,gate", CASES)
@pytest.mark.parametrize("token_major", [False, True])
def test_forward_in_runs(B, H, N, dk, dv, gate, token_major):
    print("\n[fwd runs] B=%d H=%d N=%d dk=%d dv=%d gate=%s token_major=%s" % (B, H, N, dk, dv, gate, token_major), flush=True)
    w = synth.make_sequence(3000 + N, B, H, N, dk, dv, io_dtype="bf16", gate_dtype=gate, lb=0.9, with_h0=True, with_dO=True)
    layout = binding.HGRN2_LAYOUT_BNHD if token_major else binding.HGRN2_LAYOUT_BHND
    arr = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if token_major else (lambda t: t)
    q, v, dO = (arr(dev(x, "bf16")) for x in (w.q, w.v, w.dO))
    f, h0 = arr(dev(w.f, gate)), dev(w.h0)
    o, hT = binding.hgrn2_fwd(q, f, v, h0, layout=layout)
    o2, hT2, saved = binding.hgrn2_fwd_saving(q, f, v, h0, layout=layout)
    g = binding.hgrn2_bwd_saved(q, f, v, saved, dO, layout=layout)
    torch.cuda.synchronize()
    ro, rhT = oracle.fwd(w.q, w.f, w.v, w.h0)
    check("o", host(arr(o)), ro, TOL["bf16"])
    check("hT", host(hT), rhT, TOL["bf16"])
    assert torch.equal(o, o2) and torch.equal(hT, hT2)
    for name, x, r in zip(("dq", "df", "dv"), g, oracle.bwd(w.q, w.f, w.v, w.dO, w.h0, None)):
        check(name, host(arr(x)), r, TOL["bf16"])


# 64 heads: four spans per head; lengths that make spans start and end inside sequences, cross several
# short ones, contain empty ones, and leave a sequence over three spans
@pytest.mark.parametrize("lens", [[5, 700, 64, 0, 1], [64, 64, 64, 64, 64, 64, 64, 65], [0, 30, 200], [1, 0, 0, 63, 900, 40, 130]])
@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 128)])
def test_packed_forward_in_spans(lens, dk, dv):
    print("\n[fwd spans] lens=%s dk=%d dv=%d" % (lens, dk, dv), flush=True)
    H, T, B = 64, sum(lens), len(lens)
    w = synth.make_sequence(3100 + T, 1, H, T, dk, dv, io_dtype="bf16", lb=0.9, with_dO=True)
    rng = np.random.default_rng(T)
    h0 = (0.1 * rng.standard_normal((B, H, dk, dv))).astype(np.float32)
    pk = lambda x: dev(x, "bf16")[0].permute(1, 0, 2).contiguous()
    q, f, v, dO = (pk(x) for x in (w.q, w.f, w.v, w.dO))
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), device="cuda")
    shape = binding.make_shape_varlen(q, v, f, B)
    saved = torch.full((binding.hgrn2_saved_states_varlen_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    o, hT = binding.hgrn2_fwd_varlen(q, f, v, cu, dev(h0))
    o2, hT2 = binding.hgrn2_fwd_varlen(q, f, v, cu, dev(h0), saved_states=saved)
    g = binding.hgrn2_bwd_varlen(q, f, v, dO, cu, dev(h0), saved_states=saved)
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and torch.equal(hT, hT2)
    at = 0
    for b, n in enumerate(lens):
        if n == 0:
            assert np.array_equal(host(hT[b]), h0[b].astype(np.float64))
            continue
        s = slice(at, at + n)
        at += n
        cut = lambda x: x[:, :, s]
        ro, rhT = oracle.fwd(cut(w.q), cut(w.f), cut(w.v), h0[b:b + 1])
        check("o[%d]" % b, host(o[s].permute(1, 0, 2)[None]), ro, TOL["bf16"])
        check("hT[%d]" % b, host(hT[b:b + 1]), rhT, TOL["bf16"])
        for name, x, r in zip(("dq", "df", "dv"), g, oracle.bwd(cut(w.q), cut(w.f), cut(w.v), cut(w.dO), h0[b:b + 1], None)):
            check("%s[%d]" % (name, b), host(x[s].permute(1, 0, 2)[None]), r, TOL["bf16"])


# fp32 storage: the read-out that adds up the chunks' contributions (up to 1 MB of them: 64 chunks of 64 x 64
# states, 16 of 128 x 128), its limits on either side, one chunk, a ragged last one
@pytest.mark.parametrize("B,H,N,dk,dv", [(1, 1, 256, 64, 64), (2, 3, 777, 128, 64), (1, 2, 1000, 64, 128), (1, 1, 40, 128, 128),
                                         (1, 2, 1024, 128, 128), (1, 2, 1025, 128, 128), (1, 1, 4096, 64, 64), (33, 2, 500, 64, 64)])
@pytest.mark.parametrize("states", [False, True])
def test_forward_fp32_from_contributions(B, H, N, dk, dv, states):
    print("\n[fwd f32] B=%d H=%d N=%d dk=%d dv=%d states=%s" % (B, H, N, dk, dv, states), flush=True)
    w = synth.make_sequence(3200 + N, B, H, N, dk, dv, io_dtype="f32", lb=0.9, with_h0=states)
    o, hT = binding.hgrn2_fwd(dev(w.q), dev(w.f), dev(w.v), dev(w.h0), want_hT=states)
    torch.cuda.synchronize()
    ro, rhT = oracle.fwd(w.q, w.f, w.v, w.h0)
    check("o", host(o), ro, TOL["f32"])
    if states:
        check("hT", host(hT), rhT, TOL["f32"])


# The same, where the final states just find a place beside the chunks (256 workgroups, 512 with heads of 64 x 64) and where the
# last chunks' workgroups form them, token-major; 64 x 128: 64 columns a workgroup up to 128 chunks, all columns beyond
@pytest.mark.parametrize("BH,NC,dk,dv", [(32, 3, 128, 128), (48, 2, 128, 128), (64, 3, 128, 64), (96, 2, 128, 64),
                                         (128, 3, 64, 64), (192, 2, 64, 64), (64, 3, 64, 128), (96, 2, 64, 128),
                                         (128, 1, 64, 128), (130, 1, 64, 128), (10, 13, 64, 128), (128, 1, 64, 64), (192, 1, 64, 64)])
def test_forward_fp32_final_states_beside_the_chunks(BH, NC, dk, dv):
    print("\n[fwd f32, final states] BH=%d NC=%d dk=%d dv=%d" % (BH, NC, dk, dv), flush=True)
    w = synth.make_sequence(3250 + BH, 2, BH // 2, 64 * NC - 7, dk, dv, io_dtype="f32", lb=0.5, with_h0=True)
    rows = lambda x: dev(x).permute(0, 2, 1, 3).contiguous()
    o, hT = binding.hgrn2_fwd(rows(w.q), rows(w.f), rows(w.v), dev(w.h0), layout=binding.HGRN2_LAYOUT_BNHD)
    torch.cuda.synchronize()
    ro, rhT = oracle.fwd(w.q, w.f, w.v, w.h0)
    check("o", host(o.permute(0, 2, 1, 3)), ro, TOL["f32"])
    check("hT", host(hT), rhT, TOL["f32"])


# Two light runs of 96 and 100 sequences with the gate formed in the kernels, token-major, continued from a state, the
# chunk length chosen on the device: ordinary gates (64 tokens) and gates for which shorter chunks are taken
@pytest.mark.parametrize("small", [False, True])
@pytest.mark.parametrize("B,H,N,d", [(2, 48, 330, 128), (2, 50, 330, 64)])
def test_light_runs_with_the_chunk_length_chosen_on_the_device(B, H, N, d, small):
    print("\n[fwd runs, auto] B=%d H=%d N=%d d=%d small=%d" % (B, H, N, d, small), flush=True)
    rng = np.random.default_rng(3300 + N + d)
    q, v, z = (torch.from_numpy(rng.standard_normal((B, N, H, d)).astype(np.float32)).to(torch.bfloat16) for _ in range(3))
    beta = torch.full((H, d), 0.0 if small else 0.5)
    if small:
        z = z - 5.0                      # gates near 0.007: products of 32 below 2^-100, of 8 above
    h0 = (0.1 * rng.standard_normal((B, H, d, d))).astype(np.float32)
    o, hT = binding.hgrn2_fwd_gated(q.cuda(), z.cuda(), beta.cuda(), v.cuda(), dev(h0), layout=binding.HGRN2_LAYOUT_BNHD,
                                    chunk=-1)
    torch.cuda.synchronize()
    heads = lambda x: x.permute(0, 2, 1, 3).double().numpy()
    f = heads(beta.double()[None, None] + (1.0 - beta.double()[None, None]) * torch.sigmoid(z.double()))
    ro, rhT = oracle.fwd(heads(q), f, heads(v), h0)
    check("o", host(o.permute(0, 2, 1, 3)), ro, TOL["bf16"])
    check("hT", host(hT), rhT, TOL["bf16"])
