"""The reverse walk at the edges of its tiles: sequence lengths around the 32-row tiles and the 64-row chunks, every
head-dimension pair, both layouts, gates in bf16 and fp32 and formed in the walk, chunks of 64 and 16 tokens, equal
lengths and the same lengths packed (a ragged chunk's rows then lie next to another sequence's).  Compared with the fp64
oracle: max|x-y|/max|y| <= 2e-2 per tensor (bf16 storage).  And tensors that start at an odd element: bit for bit the results of
aligned ones."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_07904_amd import binding, synth
from gpu_util import TOL, check, dev, host

pytestmark = pytest.mark.gpu
BNHD = binding.HGRN2_LAYOUT_BNHD
EDGES = [1, 4, 31, 32, 33, 63, 64, 65, 96, 129]


def make(N, dk, dv, gate, gated, seed):
    w = synth.make_sequence(seed + N, 1, 2, N, dk, dv, io_dtype="bf16", gate_dtype=gate, lb=0.4, with_dO=True)
    z = synth.bf16_round(np.random.default_rng(seed + 7 * N).standard_normal((1, 2, N, dk)).astype(np.float32))
    return w, z if gated else w.f


def reference(w, f, beta):
    if beta is None:
        dq, df, dv, _ = oracle.bwd(w.q, f, w.v, w.dO)
        return dq, df, dv, None
    dq, df, db, dv, _ = oracle.bwd_gated(w.q, f, beta, w.v, w.dO)
    return dq, df, dv, db


@pytest.mark.parametrize("dk,dv,layout,gate,gated,chunk", [
    (128, 128, 0, "bf16", False, 0), (128, 128, 1, "f32", False, 0), (128, 128, 1, "bf16", True, 0), (128, 128, 0, "bf16", False, 16),
    (64, 64, 0, "f32", True, 0), (64, 64, 1, "bf16", False, 0), (128, 64, 1, "bf16", True, 0), (64, 128, 0, "f32", False, 0),
])
def test_walk_at_tile_edges(dk, dv, layout, gate, gated, chunk):
    beta = np.random.default_rng(5).uniform(0.2, 0.9, size=(2, dk)).astype(np.float32) if gated else None
    bd = torch.from_numpy(beta).cuda() if gated else None
    put = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == BNHD else (lambda t: t)
    get = (lambda t: host(t.permute(0, 2, 1, 3))) if layout == BNHD else host
    for N in EDGES:
        print("[walk] dk=%d dv=%d N=%d chunk=%d" % (dk, dv, N, chunk), flush=True)
        w, f = make(N, dk, dv, gate, gated, 7100)
        q, fd, v, dO = put(dev(w.q, "bf16")), put(dev(f, gate)), put(dev(w.v, "bf16")), put(dev(w.dO, "bf16"))
        _, _, saved = binding.hgrn2_fwd_saving(q, fd, v, beta=bd, want_hT=False, layout=layout, chunk=chunk)
        g = binding.hgrn2_bwd_saved(q, fd, v, saved, dO, beta=bd, layout=layout, chunk=chunk)
        rq, rf, rv, rb = reference(w, f, beta)
        for name, x, r in zip(("dq", "df", "dv"), g[:3], (rq, rf, rv)):
            check(name, get(x), r, TOL["bf16"])
        if gated:
            check("dbeta", host(g[-1]), rb, TOL["bf16"])


@pytest.mark.parametrize("dk,dv,layout,gate,gated,chunk", [
    (64, 64, 1, "bf16", True, 16), (128, 64, 0, "f32", False, 32), (64, 128, 0, "bf16", True, 32), (128, 128, 1, "f32", True, 16)])
def test_fine_chunks_at_tile_edges(dk, dv, layout, gate, gated, chunk):
    test_walk_at_tile_edges(dk, dv, layout, gate, gated, chunk)


@pytest.mark.parametrize("dk,dv,gate,gated", [(128, 128, "bf16", True), (64, 64, "f32", False), (128, 64, "bf16", False), (64, 128, "bf16", True)])
def test_packed_walk_at_tile_edges(dk, dv, gate, gated):
    beta = np.random.default_rng(6).uniform(0.2, 0.9, size=(2, dk)).astype(np.float32) if gated else None
    bd = torch.from_numpy(beta).cuda() if gated else None
    parts = [make(N, dk, dv, gate, gated, 7300) for N in EDGES]
    pack = lambda xs, dt: dev(np.concatenate([x[0].transpose(1, 0, 2) for x in xs], axis=0), dt).contiguous()
    q, v, dO = (pack([getattr(w, n) for w, _ in parts], "bf16") for n in ("q", "v", "dO"))
    f = pack([f for _, f in parts], gate)
    cu = torch.tensor(np.cumsum([0] + EDGES), dtype=torch.int32, device="cuda")
    shape = binding.make_shape_varlen(q, v, f, len(EDGES))
    saved = torch.empty(max(256, binding.hgrn2_saved_states_varlen_bytes(shape)), dtype=torch.uint8, device="cuda")
    binding.hgrn2_fwd_varlen(q, f, v, cu, beta=bd, want_hT=False, saved_states=saved)
    g = binding.hgrn2_bwd_varlen(q, f, v, dO, cu, beta=bd, saved_states=saved)
    refs = [reference(w, f_, beta) for w, f_ in parts]
    for k, name in enumerate(("dq", "df", "dv")):
        r = np.concatenate([x[k][0].transpose(1, 0, 2) for x in refs], axis=0)
        check(name, host(g[k]), r, TOL["bf16"])
    if gated:
        check("dbeta", host([x for x in g if x is not None][-1]), sum(x[3] for x in refs), TOL["bf16"])


def odd(x):
    room = torch.zeros(x.numel() + 8, dtype=x.dtype, device="cuda")
    room[1:1 + x.numel()] = x.flatten()
    return room[1:1 + x.numel()].view(x.shape)


def test_tensors_that_start_at_an_odd_element():
    B, H, N, d = 2, 2, 197, 128
    gen = torch.Generator(device="cuda").manual_seed(3)
    xs = [torch.randn(B, H, N, d, generator=gen, device="cuda") for _ in range(4)]
    xs[1] = 0.4 + 0.6 * torch.sigmoid(xs[1])
    xs = [x.bfloat16() for x in xs]

    def run(q, f, v, dO):
        o, _, saved = binding.hgrn2_fwd_saving(q, f, v, want_hT=False)
        return [o] + [x for x in binding.hgrn2_bwd_saved(q, f, v, saved, dO) if x is not None]

    for a, b in zip(run(*xs), run(*[odd(x) for x in xs])):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dk,dv,layout,gate,gated,chunk", [
    (64, 64, 1, torch.float32, True, 0), (128, 64, 1, torch.float32, False, 16), (64, 128, 0, torch.bfloat16, True, 0)])
def test_other_shapes_that_start_at_an_odd_element(dk, dv, layout, gate, gated, chunk):
    """Inputs and gradients alike, which a caller of the C ABI may place as it likes."""
    B, H, N = 2, 3, 133
    gen = torch.Generator(device="cuda").manual_seed(5)
    at = lambda d: (B, N, H, d) if layout == BNHD else (B, H, N, d)
    r = lambda d: torch.randn(at(d), generator=gen, device="cuda")
    z = r(dk)
    xs = [r(dk).bfloat16(), (z if gated else 0.4 + 0.6 * torch.sigmoid(z)).to(gate), r(dv).bfloat16(), r(dv).bfloat16()]
    beta = torch.full((H, dk), 0.3, device="cuda") if gated else None

    def run(q, f, v, dO, place):
        o, _, saved = binding.hgrn2_fwd_saving(q, f, v, beta=beta, want_hT=False, layout=layout, chunk=chunk)
        g = [place(torch.zeros_like(x, dtype=torch.bfloat16)) for x in (q, f, v)]
        out = binding.hgrn2_bwd_saved(q, f, v, saved, dO, beta=beta, layout=layout, chunk=chunk, grad_q=g[0], grad_f=g[1], grad_v=g[2])
        return [o] + [x for x in out if x is not None]

    for a, b in zip(run(*xs, lambda x: x), run(*[odd(x) for x in xs], odd)):
        assert torch.equal(a, b)
