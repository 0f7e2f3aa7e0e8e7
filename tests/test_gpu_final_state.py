"""The final state's rounding.  v is zero but for the last token of every sequence, h0 is zero, and the gates are
bf16 numbers in [0.5, 1), so that 1 - f and the final state (1 - f_N)^T v_N are exact: an implementation that rounds
the product of the gates after a token (1 for the last one) with 1 - f returns it bit for bit, one that rounds
it with a gate product of the chunk in it is off by up to 2^-9.  Over the cuts of the forward walk, sequence lengths
that end a chunk, half a chunk and neither, with kept states and without, packed batches with a document per row."""
import numpy as np
import pytest
import torch

from paper_2404_07904_amd import binding

pytestmark = pytest.mark.gpu


def inputs(seed, B, H, N, dk, dv, dtype):
    g = torch.Generator(device="cuda").manual_seed(seed)
    f = (0.5 + 0.499 * torch.rand(B, H, N, dk, generator=g, device="cuda")).to(torch.bfloat16).clamp(max=1.0 - 2.0 ** -8)
    q, v = torch.randn(B, H, N, dk, generator=g, device="cuda"), torch.zeros(B, H, N, dv, device="cuda")
    v[:, :, -1] = torch.randn(B, H, dv, generator=g, device="cuda").to(torch.bfloat16).float()
    want = (1.0 - f[:, :, -1].float())[..., None] * v[:, :, -1, None, :]
    return q.to(dtype), f.to(dtype), v.to(dtype), want


@pytest.mark.parametrize("B,H,N,dk,dv", [
    (1, 1, 64, 64, 64), (1, 2, 60, 128, 64),             # one chunk
    (4, 8, 1024, 64, 64), (1, 3, 416, 128, 128),         # light walks, halves of dv
    (5, 13, 448, 128, 128),                              # light walks, whole dv
    (1, 3, 3001, 128, 128), (1, 64, 2560, 128, 128),     # walks from zero
    (1, 2, 4500, 64, 128),                               # the same with the carry kernel
    (3, 100, 190, 64, 64), (2, 80, 256, 64, 128),        # whole sequences
])
def test_final_state_is_exact_where_the_last_tokens_share_is(B, H, N, dk, dv):
    print("\n[final state] B=%d H=%d N=%d dk=%d dv=%d" % (B, H, N, dk, dv), flush=True)
    q, f, v, want = inputs(6000 + N, B, H, N, dk, dv, torch.bfloat16)
    _, hT = binding.hgrn2_fwd(q, f, v)
    _, hT2, _ = binding.hgrn2_fwd_saving(q, f, v)
    torch.cuda.synchronize()
    assert torch.equal(hT, want) and torch.equal(hT2, want)


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 128), (128, 64), (64, 128)])
@pytest.mark.parametrize("H", [2, 64])
@pytest.mark.parametrize("lens", [[64, 64, 64, 64, 64], [700, 5, 64, 0, 1, 130], [32, 1500]])
def test_final_states_of_a_packed_batch(lens, H, dk, dv):
    print("\n[final state, packed] lens=%s H=%d dk=%d dv=%d" % (lens, H, dk, dv), flush=True)
    parts = [inputs(6100 + 7 * i + n, 1, H, n, dk, dv, torch.bfloat16) if n else None for i, n in enumerate(lens)]
    q, f, v = (torch.cat([p[k][0].permute(1, 0, 2) for p in parts if p]).contiguous() for k in range(3))
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), device="cuda")
    saved = torch.empty(binding.hgrn2_saved_states_varlen_bytes(binding.make_shape_varlen(q, v, f, len(lens))), dtype=torch.uint8, device="cuda")
    _, hT = binding.hgrn2_fwd_varlen(q, f, v, cu)
    _, hT2 = binding.hgrn2_fwd_varlen(q, f, v, cu, saved_states=saved)
    torch.cuda.synchronize()
    for i, p in enumerate(parts):
        want = p[3][0] if p else torch.zeros(H, dk, dv, device="cuda")
        assert torch.equal(hT[i], want) and torch.equal(hT2[i], want), i


# fp32 storage: the same inputs, the share exact in fp32; the read-out from contributions, on either side of its
# limits, and the sweep
@pytest.mark.parametrize("B,H,N,dk,dv", [(1, 1, 256, 64, 64), (1, 1, 40, 128, 128), (2, 3, 800, 128, 64), (1, 2, 1000, 64, 128),
                                         (1, 1, 64, 64, 64), (1, 2, 1025, 128, 128), (33, 2, 500, 64, 64)])
def test_final_state_in_fp32(B, H, N, dk, dv):
    print("\n[final state, fp32] B=%d H=%d N=%d dk=%d dv=%d" % (B, H, N, dk, dv), flush=True)
    q, f, v, want = inputs(6200 + N, B, H, N, dk, dv, torch.float32)
    _, hT = binding.hgrn2_fwd(q, f, v)
    torch.cuda.synchronize()
    assert torch.equal(hT, want)
