"""What a program that uses this library has it do: the decode step of a serving loop, the forward pass
over a prompt, the forward + backward pass of a training step (equal-length, packed and element-wise)
and the whole token mixer of one layer, each through the entry points of the binding.

A case is a dict of sizes and options (`kind` names the path).  `draw` spreads them over:
  decode    B 1..256 requests, H 1..32 heads of 64 or 128, bf16 tokens, gates bf16 or fp32, or formed
            from pre-activations
  forward   B 1..64, N 1..8192 (fp32 storage: small batches), either layout, with and without an
            initial state, final state wanted
  train     B 1..8, N 64..16384, either layout, gates given or formed in the kernels, 64 tokens per
            chunk or the chunk length chosen on the device
  packed    256..32768 tokens in documents of lognormal lengths
  hgrn1     the element-wise recurrence from its pre-activations, forward + backward
  layer     projections, recurrence and their reverse mode, 64..16384 tokens, width 256..2048
"""
import math

import torch

from paper_2404_07904_amd import binding as lib

BF16, F32 = torch.bfloat16, torch.float32


def listed():
    return [
        # one request being answered token by token: 16 heads, the layer hands over pre-activations
        dict(name="decode_single", kind="decode", B=1, H=16, dk=128, dv=128, gated=True, gate="bf16"),
        # a full serving batch, in-place update of 256 requests' states (268 MB)
        dict(name="decode_batch", kind="decode", B=256, H=16, dk=128, dv=128, gated=False, gate="bf16"),
        # the fp32 path at the size a test or a numerical experiment uses it
        dict(name="forward_f32_small", kind="forward", B=1, H=1, N=256, dk=64, dv=64, io="f32", gate="f32", lb=0.5,
             gated=False, token_major=False, h0=False, chunk=0),
        # a batch of heads of 64, continued from a state
        dict(name="forward_heads64", kind="forward", B=4, H=8, N=1024, dk=64, dv=64, io="bf16", gate="bf16", lb=0.45,
             gated=False, token_major=False, h0=True, chunk=0),
        # one prompt of odd length, as the projections write it, before decoding starts
        dict(name="prefill_prompt", kind="forward", B=1, H=16, N=777, dk=128, dv=128, io="bf16", gate="bf16", lb=0.5,
             gated=True, token_major=True, h0=False, chunk=0),
        # prefill of a large batch
        dict(name="prefill_batch", kind="forward", B=32, H=16, N=2048, dk=128, dv=128, io="bf16", gate="bf16", lb=0.5,
             gated=False, token_major=False, h0=False, chunk=0),
        # the training step of a middle layer: the headline shape
        dict(name="train_layer", kind="train", B=8, H=16, N=2048, dk=128, dv=128, gate="bf16", lb=0.5, gated=False,
             token_major=False, chunk=0),
        # the same width cut into heads of 64, ragged length, gates of the first layer (no lower bound), which a
        # program hands over with the chunk length left to the device
        dict(name="train_heads64", kind="train", B=8, H=32, N=2000, dk=64, dv=64, gate="bf16", lb=0.0, gated=True,
             token_major=True, chunk=-1),
        # few long sequences with gates near one (kept in fp32: bf16 has three values there)
        dict(name="train_long", kind="train", B=2, H=16, N=16384, dk=128, dv=128, gate="f32", lb=0.99, gated=False,
             token_major=False, chunk=0),
        # documents packed along the token axis: 21 of them, 68 to 3592 tokens long
        dict(name="train_packed", kind="packed", T=16384, docs=21, H=16, dk=128, dv=128, gate="bf16", lb=0.5, gated=True),
        # the element-wise recurrence at the same width, with its activations
        dict(name="train_hgrn1", kind="hgrn1", B=8, N=2048, d=2048, lb=0.5),
        # the token mixer of a layer: projections, gate, recurrence, and the reverse mode of all three
        dict(name="train_token_mixer", kind="layer", B=8, N=2048, d=2048, head=128, lb=0.5),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "forward", "forward", "train", "train", "packed", "hgrn1", "layer"])
    lb = rng.choice([0.0, 0.25, 0.5, 0.75, 23 / 24])
    if kind == "decode":
        return dict(kind=kind, B=_log_int(rng, 1, 256), H=_log_int(rng, 1, 32), dk=rng.choice([64, 128]),
                    dv=rng.choice([64, 128]), gated=rng.random() < 0.5, gate=rng.choice(["bf16", "bf16", "f32"]))
    if kind == "hgrn1":
        d = 64 * _log_int(rng, 2, 48)
        B = _log_int(rng, 1, 16)
        return dict(kind=kind, B=B, N=_log_int(rng, 16, max(16, min(8192, (1 << 25) // (B * d)))), d=d, lb=lb)
    if kind == "layer":
        d = 256 * _log_int(rng, 1, 8)
        B = _log_int(rng, 1, 8)
        return dict(kind=kind, B=B, N=_log_int(rng, 64, 16384 // B), d=d, head=rng.choice([64, 128]), lb=lb)
    H = _log_int(rng, 1, 32)
    dk, dv = rng.choice([(64, 64), (128, 128), (128, 128), (128, 128), (128, 64), (64, 128)])
    gated, gate = rng.random() < 0.5, rng.choice(["bf16", "bf16", "f32"])
    wide = H * max(dk, dv)
    if kind == "packed":
        T = _log_int(rng, 256, min(32768, (1 << 25) // wide))
        return dict(kind=kind, T=T, docs=_log_int(rng, 1, max(2, T // 128)), H=H, dk=dk, dv=dv, gate=gate, lb=lb, gated=gated)
    chunk = rng.choice([0, 0, 0, -1])
    if kind == "train":
        B = _log_int(rng, 1, 8)
        return dict(kind=kind, B=B, H=H, N=_log_int(rng, 64, max(64, min(16384, (1 << 25) // (wide * B)))), dk=dk, dv=dv,
                    gate=gate, lb=lb, gated=gated, token_major=rng.random() < 0.5, chunk=chunk)
    f32 = rng.random() < 0.25
    B = _log_int(rng, 1, 4 if f32 else 64)
    room = (1 << (20 if f32 else 26)) // (wide * B)
    return dict(kind=kind, B=B, H=H, N=_log_int(rng, 1, max(1, min(8192, room))), dk=dk, dv=dv, io="f32" if f32 else "bf16",
                gate="f32" if f32 else gate, lb=lb, gated=gated, token_major=rng.random() < 0.5, h0=rng.random() < 0.3,
                chunk=chunk)


def _lengths(total, docs):
    """Lengths of `docs` documents that fill `total` tokens: the quantiles of a lognormal with sigma 1, in an
    order that mixes short and long ones.  Sizes are part of the case, so no seed enters."""
    p = [(i + 0.5) / docs for i in range(docs)]
    w = torch.exp(torch.erfinv(2.0 * torch.tensor(p, dtype=torch.float64) - 1.0) * math.sqrt(2.0)).tolist()
    step = next(s for s in range(max(1, int(docs * 0.618)), 2 * docs + 2) if math.gcd(s, docs) == 1)
    w = [w[(i * step) % docs] for i in range(docs)]
    ends, run = [0], 0.0
    for x in w:
        run += x
        ends.append(int(round(total * run / sum(w))))
    ends[-1] = total
    return ends


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)

    def normal(*shape, dtype=BF16, std=1.0):
        return (std * torch.randn(shape, generator=gen, device=dev)).to(dtype)

    kind = case["kind"]
    s = dict(case)
    if kind == "layer":
        B, N, d, head = case["B"], case["N"], case["d"], case["head"]
        s.update(x=normal(B, N, d), w3=normal(3 * d, d, std=d ** -0.5), b3=normal(3 * d, dtype=F32, std=0.5),
                 grad_y=normal(B, N, d // head, head))
        s["beta"] = torch.full((d // head, head), case["lb"], dtype=F32, device=dev)
        return s
    if kind == "hgrn1":
        B, N, d = case["B"], case["N"], case["d"]
        s.update(zf=normal(B, N, d), zi=normal(B, N, d), zo=normal(B, N, d), grad_y=normal(B, N, d))
        s["beta"] = torch.full((d,), case["lb"], dtype=F32, device=dev)
        s["workspace"] = torch.empty(max(256, lib.hgrn1_workspace_bytes(B, N, d)), dtype=torch.uint8, device=dev)
        return s
    H, dk, dv = case["H"], case["dk"], case["dv"]
    if kind == "decode":
        at_k, at_v, lb, io = (case["B"], H, dk), (case["B"], H, dv), 0.9, BF16
        s["state"] = normal(case["B"], H, dk, dv, dtype=F32, std=0.1)
    elif kind == "packed":
        at_k, at_v, lb, io = (case["T"], H, dk), (case["T"], H, dv), case["lb"], BF16
        s["cu_seqlens"] = torch.tensor(_lengths(case["T"], case["docs"]), dtype=torch.int32, device=dev)
    else:
        rows = (case["B"], case["N"], H) if case["token_major"] else (case["B"], H, case["N"])
        at_k, at_v, lb, io = rows + (dk,), rows + (dv,), case["lb"], F32 if case.get("io") == "f32" else BF16
        s["layout"] = lib.HGRN2_LAYOUT_BNHD if case["token_major"] else lib.HGRN2_LAYOUT_BHND
        s["h0"] = normal(case["B"], H, dk, dv, dtype=F32, std=0.1) if case.get("h0") else None
    gate = F32 if case["gate"] == "f32" else BF16
    z = normal(*at_k, dtype=F32)
    s["f"] = (z if case["gated"] else lb + (1.0 - lb) * torch.sigmoid(z)).to(gate)
    s["beta"] = torch.full((H, dk), lb, dtype=F32, device=dev) if case["gated"] else None
    s["q"], s["v"] = normal(*at_k, dtype=io), normal(*at_v, dtype=io)
    if kind in ("train", "packed"):
        s["grad_o"] = normal(*at_v)
    if kind == "packed":
        shape = lib.make_shape_varlen(s["q"], s["v"], s["f"], case["docs"])
        s["saved"] = torch.empty(max(256, lib.hgrn2_saved_states_varlen_bytes(shape)), dtype=torch.uint8, device=dev)
    return s


def run(s):
    kind = s["kind"]
    if kind == "decode":
        if s["gated"]:
            o = lib.hgrn2_step_gated(s["q"], s["f"], s["beta"], s["v"], s["state"])
        else:
            o = lib.hgrn2_step(s["q"], s["f"], s["v"], s["state"])
        return {"o": o, "state": s["state"]}
    if kind == "forward":
        if s["gated"]:
            o, hT = lib.hgrn2_fwd_gated(s["q"], s["f"], s["beta"], s["v"], s["h0"], layout=s["layout"], chunk=s["chunk"])
        else:
            o, hT = lib.hgrn2_fwd(s["q"], s["f"], s["v"], s["h0"], layout=s["layout"], chunk=s["chunk"])
        return {"o": o, "hT": hT}
    if kind == "train":
        o, _, saved = lib.hgrn2_fwd_saving(s["q"], s["f"], s["v"], beta=s["beta"], want_hT=False, layout=s["layout"],
                                           chunk=s["chunk"])
        g = lib.hgrn2_bwd_saved(s["q"], s["f"], s["v"], saved, s["grad_o"], beta=s["beta"], layout=s["layout"],
                                chunk=s["chunk"])
        return {"o": o, "grads": [x for x in g if x is not None]}
    if kind == "packed":
        o, _ = lib.hgrn2_fwd_varlen(s["q"], s["f"], s["v"], s["cu_seqlens"], beta=s["beta"], want_hT=False,
                                    saved_states=s["saved"])
        g = lib.hgrn2_bwd_varlen(s["q"], s["f"], s["v"], s["grad_o"], s["cu_seqlens"], beta=s["beta"],
                                 saved_states=s["saved"])
        return {"o": o, "grads": [x for x in g if x is not None]}
    if kind == "hgrn1":
        y, _ = lib.hgrn1_fwd_act(s["zf"], s["zi"], s["zo"], s["beta"], want_hN=False, workspace=s["workspace"])
        g = lib.hgrn1_bwd_act(s["zf"], s["zi"], s["zo"], s["beta"], s["grad_y"], workspace=s["workspace"], saved=True)
        return {"y": y, "grads": [x for x in g if x is not None]}
    # layer: Eq. 1 -> Eq. 2 -> Eq. 3 and back
    B, N, d = s["x"].shape
    heads = (B, N, d // s["head"], s["head"])
    z, v, q, av = lib.hgru2_proj_fwd(s["x"], s["w3"], s["b3"])
    z4, v4, q4 = z.view(heads), v.view(heads), q.view(heads)
    y, _, saved = lib.hgrn2_fwd_saving(q4, z4, v4, beta=s["beta"], want_hT=False, layout=lib.HGRN2_LAYOUT_BNHD)
    gq, gz, gv, _, gbeta = lib.hgrn2_bwd_saved(q4, z4, v4, saved, s["grad_y"], beta=s["beta"], layout=lib.HGRN2_LAYOUT_BNHD)
    gx, gw, gb = lib.hgru2_proj_bwd(s["x"], s["w3"], q, av, gz.view(B, N, d), gv.view(B, N, d), gq.view(B, N, d))
    return {"y": y, "grad_x": gx, "grad_w3": gw, "grad_b3": gb, "grad_beta": gbeta}


def work(case):
    """Inputs read once, outputs written once; flops of Eq. 3 as written (rank-1 update and read-out per token
    forward, the three products and the state gradient's update backward) and of the projections' products."""
    kind = case["kind"]
    if kind == "layer":
        M, d = case["B"] * case["N"], case["d"]
        rec = 12 * M * d * case["head"]
        # x, grad_y, y, grad_x in bf16; weights bf16 in, their gradients fp32 out (biases and beta the same way)
        return {"bytes": 8 * M * d + 18 * d * d + 8 * 4 * d, "flops": 18 * M * d * d + rec}
    if kind == "hgrn1":
        n = case["B"] * case["N"] * case["d"]
        # zf, zi, zo, grad_y in; y and three gradients out
        return {"bytes": 16 * n + 8 * case["d"], "flops": 20 * n}
    dk, dv, H = case["dk"], case["dv"], case["H"]
    ge = 4 if case["gate"] == "f32" else 2
    if kind == "decode":
        n = case["B"] * H
        return {"bytes": n * (8 * dk * dv + (2 + ge) * dk + 4 * dv), "flops": 5 * n * dk * dv}
    io = 4 if case.get("io") == "f32" else 2
    tokens = case["T"] if kind == "packed" else case["B"] * case["N"]
    n = tokens * H
    if kind == "forward":
        states = case["B"] * H * dk * dv * 4 * (2 if case["h0"] else 1)
        return {"bytes": n * ((io + ge) * dk + 2 * io * dv) + states, "flops": 4 * n * dk * dv}
    # q, f, v, grad_o in; o, grad_q, grad_f, grad_v out
    return {"bytes": n * ((6 + ge) * dk + 8 * dv), "flops": 12 * n * dk * dv}


def tolerance(case):
    if case["kind"] == "decode":
        return {"rel": 4e-3}          # fp32 arithmetic, the token's output rounded to bf16
    if case.get("io") == "f32":
        return {"rel": 1e-5}          # fp32 throughout
    return {"rel": 1e-2}              # bf16 operands, fp32 accumulation
