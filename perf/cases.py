"""The work a user of this package has it do, as cases that can be timed and compared.

A case is one layer call of a model on pixel tokens:

* ``forward``: inference, ``llsa.forward`` alone;
* ``step``: training, ``llsa.forward`` followed by ``llsa.backward`` on the same workspace;
* ``layer``: inference with the glue in front of the layer fused in (QK-Norm, RoPE and pooling in
  ``llsa.qknorm_rope_pool``, then ``llsa.forward_pooled``).

A program keeps the plan, the workspace and the output buffers of a layer from step to step, so ``prepare`` makes them.
"""
import math

import torch

from paper_2512_16615_amd import inputs, llsa


def _case(name, mode, heads, N, d=64, B=16, K=8, L=3, dtype="bf16", kind="smooth", batch=1, repool=0):
    return dict(name=name, mode=mode, dtype=dtype, kind=kind, batch=batch, heads=heads, N=N, d=d, B=B, K=K, L=L, repool=repool)


def listed():
    return [
        # the smallest layer: one fp32 head of a 16 x 16 grid, as in a unit test or a toy training run; launches only
        _case("tiny_fp32_step", "step", 1, 256, d=32, B=4, K=2, L=3, dtype="f32", kind="gaussian"),
        # 64 x 64 tokens, 16 heads: the low resolution a model is trained on first, and sampled at: latency-bound
        _case("n4096_step", "step", 16, 4096, L=2),
        _case("n4096_forward", "forward", 16, 4096, L=2),
        # 52 x 52 tokens: a grid that is a multiple of the block and of nothing larger, one coarse level of 169 tokens
        _case("ragged_n2704_step", "step", 16, 2704, L=1),
        # the same layer in fp32, for debugging a training run or checking the bf16 one
        _case("fp32_n4096_step", "step", 16, 4096, L=2, dtype="f32"),
        # 128 x 128 tokens, batch 2
        _case("n16384_step", "step", 16, 16384, batch=2),
        # sampling at 128 x 128 with QK-Norm and RoPE in front of the attention
        _case("n16384_layer", "layer", 16, 16384, batch=2),
        # 256 x 256 tokens, the resolution the method is for: sampling and training
        _case("n65536_forward", "forward", 16, 65536),
        _case("n65536_step", "step", 16, 65536),
        # the same grid with two coarse levels (the dense level has 256 tokens), one workspace shared by all layers of the
        # model, so that backward pools again
        _case("n65536_L2_step", "step", 16, 65536, L=2, repool=1),
        # the same grid in blocks of 64 tokens
        _case("n65536_B64_step", "step", 16, 65536, B=64, K=8, L=2),
        # 512 x 512 tokens, wide heads, twice the picks: the longest sequence
        _case("n262144_d128_step", "step", 8, 262144, d=128, K=16, L=4),
    ]


def _gathered(c):
    """Tokens one query attends to: K_l blocks of every sparse level and the whole coarsest level."""
    n = [c["N"] // c["B"] ** l for l in range(c["L"] + 1)]
    return sum(min(c["K"], n[l + 1]) * c["B"] for l in range(c["L"])) + n[c["L"]]


def _cost(c):
    return c["batch"] * c["heads"] * c["N"] * c["d"] * _gathered(c)


def draw(rng):
    """fp32: 256 to 4096 tokens of small heads; bf16: 1024 to 262144 tokens in blocks of 16, 32 or 64, coarsest level of 2 to
    400 tokens; no more work than half of the largest listed case of the type, or, with one coarse level, than the listed one."""
    by_name = {c["name"]: c for c in listed()}
    while True:
        mode = rng.choice(["forward", "step", "step", "layer"])
        kind = rng.choice(["smooth", "smooth", "smooth", "gaussian"])
        if rng.random() < 0.15:
            dtype, d, B = "f32", rng.choice([32, 64]), rng.choice([4, 16])
            K, target = rng.choice([2, 4, 8]), 2.0 ** rng.uniform(8, 12)
            most = _cost(by_name["fp32_n4096_step"]) / 2
        else:
            dtype, d, B = "bf16", rng.choice([64, 64, 64, 128]), rng.choice([16, 16, 16, 16, 32, 64])
            K, target = rng.choice([4, 6, 8, 8, 12, 16] if B == 16 else [2, 4, 8]), 2.0 ** rng.uniform(10, 18)
            most = _cost(by_name["n262144_d128_step"]) / 2
        deep = [l for l in range(1, 5) if 2 <= target / B ** l <= 400]
        if not deep:
            continue
        L = rng.choice(deep)
        if L == 1:
            most = min(most, _cost(by_name["ragged_n2704_step"]))
        N = round(target / B ** L) * B ** L
        batch, heads = rng.choice([1, 1, 2]), rng.choice([1, 2, 3, 4, 6, 8, 12, 16])
        c = _case("", mode, heads, N, d=d, B=B, K=K, L=L, dtype=dtype, kind=kind, batch=batch, repool=rng.choice([0, 0, 1]))
        if _cost(c) <= most:
            del c["name"]
            return c


def _field(c, gen, grid):
    """One tensor [batch, heads, N, d]: i.i.d. N(0, 1), or per channel a sum of 8 low-frequency sinusoids over the pixel grid
    plus 0.1 N(0, 1) (the stand-in for image activations that ``inputs.smooth_head`` describes), made on the GPU."""
    bh, N, d = c["batch"] * c["heads"], c["N"], c["d"]
    x = torch.randn(bh, N, d, generator=gen, device="cuda")
    if grid is not None:
        H, W = grid
        f = torch.randint(0, 4, (2, bh, d, 8), generator=gen, device="cuda").float()
        f[1] += (f.sum(0) == 0).float()
        phi = 2 * math.pi * torch.rand(bh, d, 8, generator=gen, device="cuda")
        amp = 0.5 * torch.randn(bh, d, 8, generator=gen, device="cuda")
        ay = f[0][:, :, None, :] * (torch.arange(H, device="cuda") * (2 * math.pi / H))[:, None] + phi[:, :, None, :]
        bx = f[1][..., None] * (torch.arange(W, device="cuda") * (2 * math.pi / W))
        rows = torch.cat([amp[:, :, None, :] * ay.sin(), amp[:, :, None, :] * ay.cos()], dim=3)      # [bh, d, H, 16]
        cols = torch.cat([bx.cos(), bx.sin()], dim=2)                                                # [bh, d, 16, W]
        smooth = torch.matmul(rows, cols).view(bh, d, N)
        x.mul_(0.1).add_(smooth.transpose(1, 2))
    dtype = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    return x.view(c["batch"], c["heads"], N, d).to(dtype)


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    grid = None
    if c["kind"] == "smooth":
        h = next(h for h in range(math.isqrt(c["N"]), 0, -1) if c["N"] % h == 0)
        grid = (h, c["N"] // h)
    s = {"mode": c["mode"]}
    s["Q"], s["K"], s["V"] = (_field(c, gen, grid) for _ in range(3))
    s["plan"] = llsa.Plan(c["batch"], c["heads"], c["N"], c["d"], c["B"], c["K"], c["L"],
                          dtype=llsa.F32 if c["dtype"] == "f32" else llsa.BF16, bwd_repool=c["repool"])
    s["ws"] = s["plan"].alloc_workspace(c["mode"] == "step")
    s["idx"] = s["plan"].alloc_indices()
    s["O"] = torch.empty_like(s["Q"])
    s["LSE"] = torch.empty(c["batch"], c["heads"], c["N"], dtype=torch.float32, device="cuda")
    if c["mode"] == "step":
        s["dO"] = _field(c, gen, None)
        s["dQ"], s["dK"], s["dV"] = (torch.empty_like(s["Q"]) for _ in range(3))
    if c["mode"] == "layer":
        s["cos"], s["sin"] = (torch.from_numpy(t).cuda() for t in inputs.rope_tables(c["N"], c["d"]))
        s["gq"], s["gk"] = (1.0 + 0.1 * torch.randn(c["d"], generator=gen, device="cuda") for _ in range(2))
    return s


def run(s):
    p = s["plan"]
    if s["mode"] == "layer":
        Q, K, ws = llsa.qknorm_rope_pool(p, s["Q"], s["K"], s["V"], s["gq"], s["gk"], s["cos"], s["sin"], workspace=s["ws"])
        O, LSE, idx = llsa.forward_pooled(p, Q, K, s["V"], ws, s["O"], s["LSE"], s["idx"])
        return {"Q": Q, "K": K, "O": O, "LSE": LSE, "idx": idx}
    O, LSE, idx, ws = llsa.forward(p, s["Q"], s["K"], s["V"], s["O"], s["LSE"], s["idx"], s["ws"])
    out = {"O": O, "LSE": LSE, "idx": idx}
    if s["mode"] == "step":
        out["dQ"], out["dK"], out["dV"] = llsa.backward(p, s["Q"], s["K"], s["V"], O, LSE, idx, s["dO"], ws, s["dQ"], s["dK"], s["dV"])
    return out


def work(case):
    c = case
    elt = 4 if c["dtype"] == "f32" else 2
    bh, N, d, B, K, L = c["batch"] * c["heads"], c["N"], c["d"], c["B"], c["K"], c["L"]
    tensor = bh * N * d * elt
    n = [N // B ** l for l in range(L + 1)]
    lists = sum(n[l + 1] * min(K, n[l + 1]) for l in range(L)) * bh
    scores = sum(n[l] * (n[l] if l == L else min(K, n[l + 1]) * B) for l in range(1, L + 1)) * bh
    # Q, K, V in; O, the logsumexp and the lists out.  Two products per gathered token, one per selection candidate.
    data, flops = 4 * tensor + 4 * bh * N + 4 * lists, 4.0 * d * _gathered(c) * N * bh + 2.0 * d * scores
    if c["mode"] == "step":                # dO in; dQ, dK, dV out.  Five more products per gathered token.
        data, flops = data + 4 * tensor, flops + 10.0 * d * _gathered(c) * N * bh
    if c["mode"] == "layer":               # the cosine and sine tables in; the normalised, rotated Q and K out
        data, flops = data + 2 * tensor + 4 * N * d, flops + 20.0 * bh * N * d
    return {"bytes": data, "flops": flops}


def tolerance(case):
    # The lists are exact: scores are fp32 sums in a stated order.  bf16 rounds every output once, and P and dS once
    # before they are multiplied; the gradients are sums that cancel in part.
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 4e-4, "differ": 0.0}
    return {"rel": 1e-2, "max": 0.2, "differ": 0.0}
