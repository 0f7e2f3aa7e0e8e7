"""Input side of the HGRU2 token mixer (Eq. 1) on the GPU -- hgru2_proj_fwd / hgru2_proj_bwd, the bf16
matrix product with bias and activation in its epilogue -- against the fp64 oracle, alone and as
the layer Eq. 1 -> Eq. 2 -> Eq. 3 (projection, hgrn2_fwd_gated on its token-major outputs, and the
whole reverse mode).  Inputs are rounded to bf16 once and the oracle sees the rounded values.
Tolerance: max|x-y|/max|y| <= 2e-2 per tensor (bf16 storage, fp32 accumulation)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2404_07904_amd import binding, synth
from gpu_util import TOL, check, dev, host

pytestmark = pytest.mark.gpu
BNHD = binding.HGRN2_LAYOUT_BNHD


def weights(seed, d):
    rng = np.random.default_rng(seed)
    w3 = synth.bf16_round((rng.standard_normal((3 * d, d)) / np.sqrt(d)).astype(np.float32))
    b3 = (0.5 * rng.standard_normal(3 * d)).astype(np.float32)
    return w3, b3


def split(w3, b3, d):
    return w3[:d], w3[d:2 * d], w3[2 * d:], b3[:d], b3[d:2 * d], b3[2 * d:]


@pytest.mark.parametrize("B,N,d", [(1, 256, 256), (3, 77, 256), (2, 300, 512), (1, 1, 256), (4, 129, 1024),
                                   (2, 160, 512), (1, 96, 1024), (1, 64, 3072)])   # whole 64-token steps of the dW3 product; a width whose dW3 takes 256-row tiles
def test_proj_fwd_bwd(B, N, d):
    print("\n[proj] B=%d N=%d d=%d" % (B, N, d), flush=True)
    rng = np.random.default_rng(9200 + N + d)
    x = synth.bf16_round(rng.standard_normal((B, N, d)).astype(np.float32))
    w3, b3 = weights(9201 + d, d)
    gz, gv, gq = (synth.bf16_round(rng.standard_normal((B, N, d)).astype(np.float32)) for _ in range(3))
    xd, wd, bd = dev(x, "bf16"), dev(w3, "bf16"), dev(b3)
    z, v, q, av = binding.hgru2_proj_fwd(xd, wd, bd)
    dx, dw, db = binding.hgru2_proj_bwd(xd, wd, q, av, dev(gz, "bf16"), dev(gv, "bf16"), dev(gq, "bf16"))
    torch.cuda.synchronize()
    U, V, W, bu, bv, bw = split(w3, b3, d)
    rz, ri, ro = oracle.hgru2_proj(x, U, V, W, bu, bv, bw)
    tol = TOL["bf16"]
    check("z", host(z), rz, tol); check("v", host(v), ri, tol); check("q", host(q), ro, tol)
    check("av", host(av), x.astype(np.float64) @ V.astype(np.float64).T + bv, tol)
    rdx, rdU, rdV, rdW, rbu, rbv, rbw = oracle.hgru2_proj_bwd(x, U, V, W, bu, bv, bw, gz, gv, gq)
    check("dx", host(dx), rdx, tol)
    check("dw3", host(dw), np.concatenate([rdU, rdV, rdW], axis=0), tol)
    check("db3", host(db), np.concatenate([rbu, rbv, rbw]), tol)


def test_proj_without_av_and_empty():
    d = 256
    w3, b3 = weights(9300, d)
    x = synth.bf16_round(np.random.default_rng(9301).standard_normal((2, 40, d)).astype(np.float32))
    z, v, q, av = binding.hgru2_proj_fwd(dev(x, "bf16"), dev(w3, "bf16"), dev(b3), keep_av=False)
    z2, v2, q2, _ = binding.hgru2_proj_fwd(dev(x, "bf16"), dev(w3, "bf16"), dev(b3))
    torch.cuda.synchronize()
    assert av is None and torch.equal(z, z2) and torch.equal(v, v2) and torch.equal(q, q2)
    e = torch.empty((0, d), dtype=torch.bfloat16, device="cuda")
    binding.hgru2_proj_fwd(e, dev(w3, "bf16"), dev(b3))
    dx, dw, db = binding.hgru2_proj_bwd(e, dev(w3, "bf16"), e, e, e, e, e)
    torch.cuda.synchronize()
    assert float(dw.abs().max()) == 0.0 and float(db.abs().max()) == 0.0
    with pytest.raises(binding.Hgrn2Error) as err:
        binding.hgru2_proj_fwd(torch.zeros((4, 192), dtype=torch.bfloat16, device="cuda"),
                               torch.zeros((576, 192), dtype=torch.bfloat16, device="cuda"), torch.zeros(576, device="cuda"))
    assert err.value.status == 3


# The element-wise pass takes 16-byte vectors of aligned arrays and pairs of others: rows of a part, of a
# batch of loads and of a block of 128, one less and one more.  dx and dW3 follow from the same bf16 values,
# so they agree bit for bit; the bias gradients are fp32 sums of M terms in another order (M 2^-24 of their sum of moduli).
@pytest.mark.parametrize("M,d", [(1, 256), (15, 256), (17, 512), (63, 256), (65, 256), (127, 256), (129, 256), (300, 768)])
def test_proj_bwd_of_unaligned_arrays(M, d):
    print("\n[proj unaligned] M=%d d=%d" % (M, d), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(9400 + M)
    rnd = lambda *n: torch.randn(n, generator=gen, device="cuda").to(torch.bfloat16)
    x, w3 = rnd(M, d), rnd(3 * d, d)
    args = [torch.sigmoid(rnd(M, d))] + [rnd(M, d) for _ in range(4)]           # q, av, grad_z, grad_v, grad_q
    moved = []
    for t in args:
        m = torch.empty(M * d + 2, dtype=torch.bfloat16, device="cuda")[2:].view(M, d)
        m.copy_(t)
        assert m.data_ptr() % 16 == 4 and t.data_ptr() % 16 == 0
        moved.append(m)
    dx, dw, db = binding.hgru2_proj_bwd(x, w3, *args)
    dx2, dw2, db2 = binding.hgru2_proj_bwd(x, w3, *moved)
    torch.cuda.synchronize()
    assert torch.equal(dx, dx2) and torch.equal(dw, dw2)
    q, av, gz, gv, gq = (t.double() for t in args)
    sg = torch.sigmoid(av)
    ref = torch.cat([gz, gv * sg * (1.0 + av * (1.0 - sg)), gq * q * (1.0 - q)], dim=1)
    bound = (M * 2.0 ** -24 + 2.0 ** -8 + 2.0 ** -18) * ref.abs().sum(0) + 1e-30       # sums; bf16 terms; sigmoid in fp32
    assert bool(((db.double() - ref.sum(0)).abs() <= bound).all())
    assert bool(((db.double() - db2.double()).abs() <= 2 * M * 2.0 ** -24 * 1.01 * ref.abs().sum(0) + 1e-30).all())


@pytest.mark.parametrize("B,N,d,H", [(2, 200, 256, 2), (1, 333, 512, 4)])
def test_layer_projection_recurrence_and_reverse_mode(B, N, d, H):
    """Eq. 1 -> Eq. 2 -> Eq. 3: projection, then hgrn2_fwd_gated on its token-major outputs (no copy in
    between), then the reverse mode back to x, the weights, the biases and beta."""
    print("\n[layer] B=%d N=%d d=%d H=%d" % (B, N, d, H), flush=True)
    dh = d // H
    rng = np.random.default_rng(9400 + d)
    x = synth.bf16_round(rng.standard_normal((B, N, d)).astype(np.float32))
    w3, b3 = weights(9401 + d, d)
    beta = rng.uniform(0.0, 0.8, size=d).astype(np.float32)
    dy = synth.bf16_round(rng.standard_normal((B, N, d)).astype(np.float32))
    h0 = (0.1 * rng.standard_normal((B, H, dh, dh))).astype(np.float32)
    dhT = (0.1 * rng.standard_normal((B, H, dh, dh))).astype(np.float32)
    xd, wd, bd = dev(x, "bf16"), dev(w3, "bf16"), dev(b3)
    betad = torch.from_numpy(beta.reshape(H, dh)).cuda()
    z, v, q, av = binding.hgru2_proj_fwd(xd, wd, bd)
    as4 = lambda t: t.view(B, N, H, dh)
    y, hT = binding.hgrn2_fwd_gated(as4(q), as4(z), betad, as4(v), dev(h0), layout=BNHD)
    gq, gz, gb, gv, gh0 = binding.hgrn2_bwd_gated(as4(q), as4(z), betad, as4(v), as4(dev(dy, "bf16")), dev(h0), dev(dhT),
                                                  want_grad_h0=True, layout=BNHD)
    dx, dw, db = binding.hgru2_proj_bwd(xd, wd, q, av, gz.view(B, N, d), gv.view(B, N, d), gq.view(B, N, d))
    torch.cuda.synchronize()
    U, V, W, bu, bv, bw = split(w3, b3, d)
    ry, rhT = oracle.hgru2_layer_fwd(x, U, V, W, bu, bv, bw, beta, H, h0)
    g = oracle.hgru2_layer_bwd(x, U, V, W, bu, bv, bw, beta, H, dy, h0, dhT)
    tol = TOL["bf16"]
    check("y", host(y).reshape(B, N, d), ry, tol); check("hT", host(hT), rhT, tol)
    check("dx", host(dx), g[0], tol)
    check("dw3", host(dw), np.concatenate([g[1], g[2], g[3]], axis=0), tol)
    check("db3", host(db), np.concatenate([g[4], g[5], g[6]]), tol)
    check("dbeta", host(gb).reshape(-1), g[7], tol); check("dh0", host(gh0), g[8], tol)


def test_proj_full_width_sampled_rows():
    """The benchmark's projection (16384 tokens, width 2048): 512 seeded rows of z, v, q against the
    oracle (each row of the product is independent of the others)."""
    M, d = 16384, 2048
    print("\n[proj] full width: M=%d d=%d" % (M, d), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(9500)
    xd = torch.randn((M, d), generator=gen, device="cuda").to(torch.bfloat16)
    w3, b3 = weights(9501, d)
    z, v, q, av = binding.hgru2_proj_fwd(xd, dev(w3, "bf16"), dev(b3))
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(9502).choice(M, 512, replace=False))
    rows[0], rows[-1] = 0, M - 1
    rt = torch.from_numpy(rows).cuda()
    xs = host(xd[rt])
    U, V, W, bu, bv, bw = split(w3, b3, d)
    rz, ri, ro = oracle.hgru2_proj(xs[None], U, V, W, bu, bv, bw)
    tol = TOL["bf16"]
    check("z", host(z[rt]), rz[0], tol); check("v", host(v[rt]), ri[0], tol); check("q", host(q[rt]), ro[0], tol)


@pytest.mark.parametrize("M,d", [(1, 256),          # one token: 63 padded ones in the product over the tokens
                                 (1500, 512),       # a padded step; 32 tokens to a workgroup of the element-wise pass
                                 (4100, 256),       # dW3 in 64 x 64 tiles, its contraction in 4 shares of 16 and 17 steps
                                 (2048, 1024),      # 128 x 128 tiles, one share
                                 (3500, 768), (4900, 512), (9984, 256),      # dW3 in 128 x 128 tiles and 2, 4, 16 shares
                                 (4097, 1280),      # 256 x 256 tiles with one row in the last; dW3 in 192 x 256, one share
                                 (5633, 1280), (14720, 1024),                # dW3 in 192 x 256 tiles and 2, 4 shares
                                 (9000, 1024)])     # dx in 256 x 256 tiles
def test_proj_tiles_and_padding(M, d):
    """Every tile size of the products and number of shares, with a remainder of tokens (tests/test_proj_plan_host.py says which
    plan each size takes): against fp32 products of the same rounded operands
    (torch), the workspace filled with NaN before; bf16 outputs to 2 units in the last place of the
    largest value, the fp32 sums to 1e-3 (see below)."""
    print("\n[proj tiles] M=%d d=%d" % (M, d), flush=True)
    g = torch.Generator(device="cuda").manual_seed(9500 + M)
    n = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    x, w3, b3 = n(M, d), (n(3 * d, d).float() / d ** 0.5).bfloat16(), torch.randn(3 * d, generator=g, device="cuda")
    gz, gv, gq = n(M, d), n(M, d), n(M, d)
    z, v, q, av = binding.hgru2_proj_fwd(x, w3, b3)
    size = binding.lib().hgru2_proj_bwd_workspace_bytes
    size.restype = ctypes.c_size_t
    ws = torch.full((size(M, d),), 255, dtype=torch.uint8, device="cuda")
    dx, dw, db = binding.hgru2_proj_bwd(x, w3, q, av, gz, gv, gq, workspace=ws)
    a, qf = av.double(), q.double()
    s = torch.sigmoid(a)
    dA = torch.cat([gz.double(), gv.double() * s * (1 + a * (1 - s)), gq.double() * qf * (1 - qf)], 1).bfloat16().double()
    pre = x.double() @ w3.double().t() + b3.double()
    rv = pre[:, d:2 * d] * torch.sigmoid(pre[:, d:2 * d])
    for name, got, ref, tol in (("z", z, pre[:, :d], 2.0 ** -7), ("av", av, pre[:, d:2 * d], 2.0 ** -7), ("v", v, rv, 2.0 ** -7),
                                ("q", q, torch.sigmoid(pre[:, 2 * d:]), 2.0 ** -7), ("dx", dx, dA @ w3.double(), 2.0 ** -7),
                                # (an element of dA may round the other way where it is formed in another order: 2^-9 of it, in a share of the elements)
                                ("dw3", dw, dA.t() @ x.double(), 1e-3), ("db3", db, dA.sum(0), 1e-3)):
        e = float((got.double() - ref).abs().max() / ref.abs().max())
        print("   %-4s %.2e" % (name, e), flush=True)
        assert e <= tol, (name, e)


@pytest.mark.parametrize("keep_av", [True, False])
@pytest.mark.parametrize("M", [14593,       # 58 x 12 tiles for 256 workgroups: two or three each; the last row of tiles has one new row
                               14848])      # the same tiles, all rows new
def test_projection_walks_tiles(M, keep_av):
    """Projections whose workgroups take several 256 x 256 tiles (the ring of operands goes on from one to the next): every output
    element against fp64 products of the same operands, and the rows of the last two tiles, some of which both compute (which of them
    stores such a row does not show, they agree), as in a call of those rows alone; nothing is written where no tile belongs (a tail
    of sentinel rows behind every output).  bf16 outputs to 2 units in the last place of the largest value, and of the two
    calls, whose fp32 sums differ in order (1e-4 covers them where a result is near zero), to one unit of each value."""
    d = 1024
    print("\n[proj walk] M=%d keep_av=%s" % (M, keep_av), flush=True)
    g = torch.Generator(device="cuda").manual_seed(9700 + M)
    x = torch.randn((M, d), generator=g, device="cuda").bfloat16()
    w3 = (torch.randn((3 * d, d), generator=g, device="cuda") / d ** 0.5).bfloat16()
    b3 = torch.randn(3 * d, generator=g, device="cuda")
    outs = [torch.full((M + 256, d), -7.0, dtype=torch.bfloat16, device="cuda") for _ in range(4)]
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = binding.lib().hgru2_proj_fwd(M, d, ptr(x), ptr(w3), ptr(b3), ptr(outs[0]), ptr(outs[1]), ptr(outs[2]),
                                      ptr(outs[3]) if keep_av else None,
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    pre = x.double() @ w3.double().t() + b3.double()
    refs = (pre[:, :d], pre[:, d:2 * d] * torch.sigmoid(pre[:, d:2 * d]), torch.sigmoid(pre[:, 2 * d:]), pre[:, d:2 * d])
    for name, got, ref in zip(("z", "v", "q", "av"), outs, refs):
        assert bool((got[M:] == -7.0).all()), name
        if name == "av" and not keep_av:
            assert bool((got == -7.0).all())
            continue
        e = float((got[:M].double() - ref).abs().max() / ref.abs().max())
        print("   %-4s %.2e" % (name, e), flush=True)
        assert e <= 2.0 ** -7, (name, e)
    few = binding.hgru2_proj_fwd(x[M - 300:].contiguous(), w3, b3)
    for name, got, small in zip(("z", "v", "q", "av"), outs, few):
        if name == "av" and not keep_av:
            continue
        a, b = got[M - 300:M].double(), small.reshape(300, d).double()
        assert bool(((a - b).abs() <= 2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 1e-4).all()), name
