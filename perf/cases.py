"""Timed cases of the WHTMix framework: what a program that uses it has it do.

A case is a dict of plain values:

    op     "mix"          one inference call of the mixer (whtmix.forward / forward_separable)
           "mix_train"    the differentiable mixer, forward and backward (whtmix_mix*)
           "block"        one inference call of the block with its projections, eqs. (1)-(4)
           "block_train"  the differentiable block, forward and backward (whtmix_block*)
    gain   "joint" (a float32 gain per frequency) or "separable" (the paper's log-gain vectors)
    dtype  "f32" or "bf16", the element type of x, y, dy, dx and the projection weights
    B, N, C   slices, tokens (any count; the transform pads it to a power of two), channels

listed() holds the cases that stand for the uses below, draw() more of the same ranges.
Calls go through paper_2607_25234_amd.whtmix (inference) and .autograd (training).
"""
from __future__ import annotations

import math

import torch

from paper_2607_25234_amd import autograd, whtmix


def _case(name, op, gain, dtype, B, N, C):
    return {"name": name, "op": op, "gain": gain, "dtype": dtype, "B": B, "N": N, "C": C}


def listed():
    return [
        # One 32x32 byte-level image: the smallest call, bound by launches.
        _case("image1k_mix", "mix", "joint", "f32", 1, 1024, 64),
        # One 384x768 stereo pair at inference, the paper's own gains: a ragged token count
        # (9216 of 16384) and a single slice, where latency and idle compute units count.
        _case("frame9k_mix_sep", "mix", "separable", "f32", 1, 9216, 64),
        # Two 512x1024 stereo pairs, float32.
        _case("stereo16k_mix", "mix", "joint", "f32", 2, 16384, 128),
        # Four 1024x2048 stereo pairs in bf16: the benchmarked workload.
        _case("stereo64k_mix", "mix", "joint", "bf16", 4, 65536, 128),
        # One 2048x4096 stereo pair: the largest single slice, with 256 channels.
        _case("stereo256k_mix", "mix", "joint", "bf16", 1, 262144, 256),
        # A training step of the mixer on a batch of 4096-byte texts, float32.
        _case("text4k_mix_train", "mix_train", "separable", "f32", 32, 4096, 64),
        # A training step of the mixer with a gain per frequency, large bf16 slices.
        _case("stereo64k_mix_train", "mix_train", "joint", "bf16", 4, 65536, 128),
        # The block at inference on one 896x1792 pair: 50176 of 65536 tokens.
        _case("frame50k_block_sep", "block", "separable", "bf16", 1, 50176, 64),
        # The block at inference on the benchmarked shape.
        _case("stereo64k_block", "block", "joint", "bf16", 4, 65536, 128),
        # A training step of the block on a batch of 32x32 images, float32.
        _case("image1k_block_train", "block_train", "separable", "f32", 64, 1024, 64),
        # A training step of the block on two 768x1536 pairs, float32: 36864 of 65536 tokens.
        _case("frame36k_block_train", "block_train", "joint", "f32", 2, 36864, 64),
        # A training step of the block on the benchmarked shape with the paper's gains.
        _case("stereo64k_block_train", "block_train", "separable", "bf16", 4, 65536, 128),
    ]


# Most elements B * N_pad * C of a drawn case, so that none costs more than the largest listed
# ones (the weight gradients of wide blocks grow with C).
def _most(op, C):
    if op == "mix":
        return 1 << 26
    if op == "block_train" and C >= 256:
        return 1 << 22
    if op == "block" and C >= 256:
        return 1 << 24
    return 1 << 25


def draw(rng):
    op = rng.choice(["mix", "mix_train", "block", "block_train"])
    C = rng.choice([32, 64, 64, 128, 128, 256])
    most = _most(op, C)
    # tokens: 256 .. 262144 over their logarithm, a third of them powers of two
    top = min(262144, most // C)
    N = int(round(math.exp(rng.uniform(math.log(256), math.log(top)))))
    if rng.random() < 1 / 3:
        N = 1 << max(8, N.bit_length() - 1)
    N = max(256, min(N, top))
    P = whtmix.padded_tokens(N)
    B = max(1, min(64, most // (P * C)))
    B = int(round(math.exp(rng.uniform(0.0, math.log(B)))))
    return {"op": op, "gain": rng.choice(["joint", "separable"]),
            "dtype": rng.choice(["f32", "bf16"]), "B": B, "N": N, "C": C}


def prepare(case, seed):
    B, N, C = case["B"], case["N"], case["C"]
    P = whtmix.padded_tokens(N)
    dev = torch.device("cuda")
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(*shape, std=1.0, dtype=torch.float32):
        return (torch.randn(*shape, generator=gen, device=dev) * std).to(dtype)

    train = case["op"].endswith("_train")
    s = {"case": case, "x": normal(B, N, C, dtype=dt)}
    if case["op"].startswith("block"):
        s["w_in"] = normal(C, C, std=C ** -0.5, dtype=dt)
        s["w_out"] = normal(C, C, std=C ** -0.5, dtype=dt)
    if case["gain"] == "joint":
        s["gain"] = torch.rand(P, C, generator=gen, device=dev) + 0.5
    else:
        s["gt"] = normal(P, std=0.3)
        s["gc"] = normal(C, std=0.3)
    if train:
        s["dy"] = normal(B, N, C, dtype=dt)
        for k in ("x", "w_in", "w_out", "gain", "gt", "gc"):
            if k in s:
                s[k].requires_grad_(True)
    return s


def run(s):
    case = s["case"]
    block = case["op"].startswith("block")
    gains = (s["gain"],) if case["gain"] == "joint" else (s["gt"], s["gc"])
    args = (s["x"], s["w_in"], *gains, s["w_out"]) if block else (s["x"], *gains)
    if not case["op"].endswith("_train"):
        if block:
            f = whtmix.module_forward if len(gains) == 1 else whtmix.module_forward_separable
        else:
            f = whtmix.forward if len(gains) == 1 else whtmix.forward_separable
        return f(*args)
    if block:
        f = autograd.whtmix_block if len(gains) == 1 else autograd.whtmix_block_separable
    else:
        f = autograd.whtmix_mix if len(gains) == 1 else autograd.whtmix_mix_separable
    y = f(*args)
    return [y.detach(), *torch.autograd.grad(y, args, s["dy"])]


def work(case):
    B, N, C = case["B"], case["N"], case["C"]
    P = whtmix.padded_tokens(N)
    size = 2 if case["dtype"] == "bf16" else 4
    train = case["op"].endswith("_train")
    block = case["op"].startswith("block")
    # x in, y out; in training dy in and dx out too; gains and weights once, and their gradients
    passes = 2 if train else 1
    gain = 4 * P * C if case["gain"] == "joint" else 4 * (P + C)
    weights = 2 * C * C * size if block else 0
    nbytes = passes * (2 * B * N * C * size + gain + weights)
    # per padded element: log2(P C) additions each way and the gain; a training step has the
    # forward's two transforms, dy's two and the gain gradient's product
    K = int(math.log2(P * C))
    flops = B * P * C * (2 * K + 1) * passes + (2 * B * P * C if train else 0)
    if block:
        flops += 2 * B * N * C * C * (6 if train else 2)
    return {"bytes": nbytes, "flops": flops}


# float32: measured against exact(), outputs are 1e-7 to 5e-7 off (2-norm), so that two correct
# implementations differ by less than 2e-6.  bf16: one rounding to nearest even of each output is
# 1.7e-3 of it (2-norm); 5e-3 allows for a few roundings that fall the other way.
def tolerance(case):
    return {"rel": 5e-3} if case["dtype"] == "bf16" else {"rel": 2e-6}


def _wht(v, dim):
    """Orthonormal Sylvester Walsh-Hadamard transform of v along dim (-1 or -2), in place of v."""
    n = v.shape[dim]
    tail = 1 if dim == -1 else v.shape[-1]
    h = 1
    while h < n:
        w = v.view(-1, 2, h * tail)
        a, b = w[:, 0], w[:, 1]
        s = a + b
        torch.sub(a, b, out=b)
        a.copy_(s)
        h *= 2
    return v.mul_(n ** -0.5)


def _pad(v, P):
    out = torch.zeros(v.shape[0], P, v.shape[2], dtype=torch.float64, device=v.device)
    out[:, :v.shape[1]] = v
    return out


def _transform(v):
    return _wht(_wht(v, -1), -2)


def exact(case, seed):
    s = prepare(case, seed)
    N = case["N"]
    P = whtmix.padded_tokens(N)
    d = {k: v.detach().double() for k, v in s.items() if k != "case"}
    block = case["op"].startswith("block")
    joint = case["gain"] == "joint"
    g = d["gain"] if joint else torch.exp(d["gt"])[:, None] * torch.exp(d["gc"])[None, :]
    z = d["x"] @ d["w_in"] if block else d["x"]
    fz = _transform(_pad(z, P))
    zp = _transform(fz * g)[:, :N].clone()
    y = zp @ d["w_out"] if block else zp
    if not case["op"].endswith("_train"):
        return y
    fd = _transform(_pad(d["dy"] @ d["w_out"].T if block else d["dy"], P))
    dg = (fz * fd).sum(0)
    dz = _transform(fd * g)[:, :N].clone()
    dgains = [dg] if joint else [(dg * g).sum(1), (dg * g).sum(0)]
    if not block:
        return [y, dz, *dgains]
    rows = lambda v: v.reshape(-1, v.shape[-1])  # noqa: E731
    dw_in = rows(d["x"]).T @ rows(dz)
    dw_out = rows(zp).T @ rows(d["dy"])
    return [y, dz @ d["w_in"].T, dw_in, *dgains, dw_out]
