"""So many heads side by side that the rows of a chunk lie gigabytes apart: the reverse walk then takes 64-bit row addresses
(csrc/walk_rows.hpp says from which stride on), and a few rows of the other kernels are more than an int apart.  The heads repeat 512 heads, so every element of every result has to be that of a
call over those alone; bf16 results to 2 units in the last place of the largest value (another instance of the kernel
may contract its sums in another way; a row that was taken for another one is off by the value itself)."""
import pytest
import torch

from paper_2404_07904_amd import binding

pytestmark = pytest.mark.gpu
BNHD = binding.HGRN2_LAYOUT_BNHD
FEW = 512


def few_heads(seed, rows, dk, dv, gate, gated):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda d: torch.randn((rows, FEW, d), generator=gen, device="cuda")
    z = r(dk)
    f = (z if gated else 0.4 + 0.6 * torch.sigmoid(z)).to(gate)
    beta = torch.rand((FEW, dk), generator=gen, device="cuda") * 0.5 + 0.3 if gated else None
    return r(dk).bfloat16(), f, r(dv).bfloat16(), r(dv).bfloat16(), beta


def same(name, far, few, times):
    """far: the heads of `few` over and over, along the axis before the last"""
    far, few = far.reshape(-1, times, FEW, far.shape[-1]), few.reshape(-1, 1, FEW, few.shape[-1])
    tol = 2.0 ** -7 * float(few.abs().max())
    assert tol > 0.0
    for i in range(far.shape[0]):
        e = (far[i].float() - few[i].float()).abs().amax()
        assert float(e) <= tol, (name, i, float(e), tol)


def room(gib):
    if torch.cuda.mem_get_info()[0] < gib * 2 ** 30:
        pytest.skip("needs %d GiB of GPU memory" % gib)


@pytest.mark.parametrize("H,dk,dv,N,gate,gated", [
    (288 * FEW, 128, 128, 64, torch.float32, False),      # a descriptor's length would be over 4 GiB
    (2048 * FEW, 64, 64, 1, torch.bfloat16, True),        # row 32, which stands for no token, would lie on row 0
    (512 * FEW, 128, 64, 66, torch.bfloat16, False),      # two chunks
    (256 * FEW, 64, 128, 3, torch.float32, True),
])
def test_backward_of_far_rows(H, dk, dv, N, gate, gated):
    room(80)
    print("\n[far rows] H=%d dk=%d dv=%d N=%d" % (H, dk, dv, N), flush=True)
    q, f, v, dO, beta = few_heads(41 + N, N, dk, dv, gate, gated)

    def run(times):
        rep = lambda x: None if x is None else x.repeat(*([1] * (x.dim() - 2)), times, 1)
        put = lambda x: rep(x).unsqueeze(0)
        a, g, b, c, be = put(q), put(f), put(v), put(dO), rep(beta)
        o, _, saved = binding.hgrn2_fwd_saving(a, g, b, beta=be, want_hT=False, layout=BNHD)
        r = [o] + [x for x in binding.hgrn2_bwd_saved(a, g, b, saved, c, beta=be, layout=BNHD) if x is not None]
        torch.cuda.synchronize()
        return r

    times = H // FEW
    few = run(1)
    far = run(times)
    assert len(far) == (5 if gated else 4)
    for name, x, y in zip(("o", "dq", "df", "dv", "dbeta"), far, few):
        same(name, x, y, times)
    del far
    torch.cuda.empty_cache()


@pytest.mark.parametrize("saved", [True, False])
def test_packed_backward_of_far_rows(saved):
    room(80)
    times, dk, dv, lens = 1024, 64, 64, [1, 0, 2]
    print("\n[far rows, packed] H=%d saved=%s" % (times * FEW, saved), flush=True)
    q, f, v, dO, beta = few_heads(43, sum(lens), dk, dv, torch.float32, True)
    cu = torch.tensor([0, 1, 1, 3], dtype=torch.int32, device="cuda")

    def run(times):
        a, g, b, c, be = (x.repeat(*([1] * (x.dim() - 2)), times, 1) for x in (q, f, v, dO, beta))
        keep = None
        if saved:
            shape = binding.make_shape_varlen(a, b, g, len(lens))
            keep = torch.empty(max(256, binding.hgrn2_saved_states_varlen_bytes(shape)), dtype=torch.uint8, device="cuda")
            binding.hgrn2_fwd_varlen(a, g, b, cu, beta=be, want_hT=False, saved_states=keep)
        r = [x for x in binding.hgrn2_bwd_varlen(a, g, b, c, cu, beta=be, saved_states=keep) if x is not None]
        torch.cuda.synchronize()
        return r

    few = run(1)
    far = run(times)
    for i, (x, y) in enumerate(zip(far, few)):
        same("grad %d" % i, x, y, times)
    del far
    torch.cuda.empty_cache()


@pytest.mark.parametrize("what,H,dk,dv,N", [
    ("fwd", 2560 * FEW, 64, 64, 16), ("fwd", 1280 * FEW, 128, 128, 8), ("f32", 2048 * FEW, 64, 64, 16), ("bwd", 2048 * FEW, 64, 64, 16)])
def test_whole_blocks_of_far_rows(what, H, dk, dv, N):
    """Rows of 320 MiB (256 in the last two) of fp32 gates, in blocks of 8 and 16 that lie inside the sequence: the forward pass, the one of
    fp32 storage (sweep and read-out, which so many heads of 64 take in bf16 too) and the stateless backward pass (sweep and reverse walk)."""
    room(160)
    print("\n[far rows, blocks] %s H=%d dk=%d dv=%d N=%d" % (what, H, dk, dv, N), flush=True)
    q, f, v, dO, _ = few_heads(47, N, dk, dv, torch.float32, False)
    if what == "f32":
        q, v = q.float(), v.float()

    def run(times):
        a, g, b, c = (x.repeat(1, times, 1).unsqueeze(0) for x in (q, f, v, dO))
        if what == "bwd":
            r = [x for x in binding.hgrn2_bwd(a, g, b, c, layout=BNHD) if x is not None]
        else:
            r = list(binding.hgrn2_fwd(a, g, b, layout=BNHD))
        torch.cuda.synchronize()
        return r

    times = H // FEW
    few = run(1)
    far = run(times)
    for i, (x, y) in enumerate(zip(far, few)):
        if x.dim() == 4 and x.shape[1] != N:          # the final state: a head's rows together
            x, y = x.reshape(1, H, dk * dv), y.reshape(1, FEW, dk * dv)
        same("%s %d" % (what, i), x, y, times)
    del far
    torch.cuda.empty_cache()
