"""Zero-padded slices whose wholly padded outer tiles are left out of the
workspace: neither stored by the first pass nor read by the middle one.  Every
call here runs after one on the same stream that leaves NaN throughout the
workspace, so a row that is read without having been written shows."""
import numpy as np
import pytest

from oracle import oracle as oracle_mod
from paper_2607_25234_amd import whtmix, workloads
from tests.gpu_util import DERIVED, device, errors, say, to_device, to_host

pytestmark = pytest.mark.gpu

# (B, N, C): five eighths of the rows kept (one real outer tile past half of them, a
# straddling tile, slice groups in the middle pass with B = 4 of 2^21), six and
# seven eighths, and all of them with one tile padded
SHAPES = [(1, 9216, 64), (2, 4097, 64), (3, 2040, 128), (1, 36864, 64), (4, 9000, 128),
          (1, 600, 128), (2, 25600, 32), (1, 700, 128), (64, 700, 64)]


@pytest.fixture(scope="module")
def dev():
    return device()


@pytest.fixture(scope="module")
def orc():
    return oracle_mod.Oracle()


def poison(B, N, C, dtype, dev, block):
    """NaN through every workspace row of this shape's calls."""
    import torch

    P = whtmix.padded_tokens(N)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.full((B, P, C), float("nan"), device=dev, dtype=tdt)
    g = torch.ones(P, C, device=dev)
    if block:
        w = torch.ones(C, C, device=dev, dtype=tdt)
        whtmix.module_forward(x, w, g, w)
        whtmix.module_backward(x, w, g, w, x)
    else:
        whtmix.forward(x, g)
        whtmix.backward(x, x, g)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_padded_rows_left_out(shape, dtype, dev, orc):
    import torch

    B, N, C = shape
    P = whtmix.padded_tokens(N)
    x, _ = workloads.draw(B, N, C, dtype, seed=700 + N)
    dy, _ = workloads.draw(B, N, C, dtype, seed=701 + N)
    _, g = workloads.draw(1, P, C, "f32", seed=702 + N)
    wi, wo = workloads.draw_weights(C, dtype, seed=703 + N)
    say(f"padding {shape} {dtype} plan={whtmix.plan_describe(B, N, C, dtype)['plan']}")
    xd, dyd = to_device(x, dtype, dev), to_device(dy, dtype, dev)
    gd = to_device(g, "f32", dev)
    wid, wod = to_device(wi, dtype, dev), to_device(wo, dtype, dev)

    def check(name, t, ref, tol):
        err = errors(to_host(t), ref)[0]
        assert err <= tol, (name, err)     # NaN fails too

    poison(B, N, C, dtype, dev, False)
    y = whtmix.forward(xd, gd, plan="three_pass")
    poison(B, N, C, dtype, dev, False)
    dx, dg = whtmix.backward(xd, dyd, gd)
    poison(B, N, C, dtype, dev, False)
    _, dg_only = whtmix.backward(xd, dyd, gd, want_dx=False)
    poison(B, N, C, dtype, dev, True)
    yb = whtmix.module_forward(xd, wid, gd, wod)
    poison(B, N, C, dtype, dev, True)
    dxb, dwi, dwo, dgb = whtmix.module_backward(xd, wid, gd, wod, dyd)
    torch.cuda.synchronize(dev)
    check("y", y, orc.whtmix(x, g), DERIVED[dtype])
    rdx, rdg = orc.whtmix_grad(x, dy, g)
    check("dx", dx, rdx, DERIVED[dtype])
    check("dg", dg, rdg, 1e-5)
    check("dg alone", dg_only, rdg, 1e-5)
    block = {"f32": 1e-5, "bf16": 4e-3}[dtype]
    check("block y", yb, orc.whtmix_module(x, wi, g, wo), block)
    ref = orc.whtmix_module_grad(x, wi, g, wo, dy)
    for name, t, r, tol in zip(["dx", "dw_in", "dw_out", "dg"], [dxb, dwi, dwo, dgb], ref,
                               [block, 1e-5, 1e-5, 1e-5]):
        check("block " + name, t, r, tol)


def test_padded_pair_tiles_left_out(dev):
    """2^16 outer tiles (one bf16 slice of 140000 x 256): against the same
    slice with its padding rows given as real zeros."""
    import torch

    N, C = 140000, 256
    P = whtmix.padded_tokens(N)
    gen = torch.Generator(device=dev).manual_seed(9)
    x = torch.zeros(1, P, C, device=dev, dtype=torch.bfloat16)
    x[:, :N] = torch.randn(1, N, C, generator=gen, device=dev)
    g = torch.rand(P, C, generator=gen, device=dev) + 0.5
    poison(1, N, C, "bf16", dev, False)
    y = whtmix.forward(x[:, :N].contiguous(), g)
    full = whtmix.forward(x, g)
    torch.cuda.synchronize(dev)
    assert torch.equal(y, full[:, :N])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 9216, 64), (2, 25600, 32), (3, 700, 128), (8, 4700, 64)],
                         ids=lambda s: "x".join(map(str, s)))
def test_padded_rows_left_out_separable(shape, dtype, dev, orc):
    """The same with the paper's log gains: the middle passes that form the log-gain
    gradients' sums themselves, and those of 2^11 tiles that leave dG to a kernel."""
    import torch

    B, N, C = shape
    P = whtmix.padded_tokens(N)
    x, _ = workloads.draw(B, N, C, dtype, seed=710 + N)
    dy, _ = workloads.draw(B, N, C, dtype, seed=711 + N)
    gt, gc = workloads.draw_log_gains(P, C, seed=712 + N)
    wi, wo = workloads.draw_weights(C, dtype, seed=713 + N)
    say(f"padding separable {shape} {dtype}")
    xd, dyd = to_device(x, dtype, dev), to_device(dy, dtype, dev)
    gtd, gcd = to_device(gt, "f32", dev), to_device(gc, "f32", dev)
    wid, wod = to_device(wi, dtype, dev), to_device(wo, dtype, dev)
    poison(B, N, C, dtype, dev, False)
    y = whtmix.forward_separable(xd, gtd, gcd, plan="three_pass")
    poison(B, N, C, dtype, dev, False)
    got = whtmix.backward_separable(xd, dyd, gtd, gcd)
    poison(B, N, C, dtype, dev, True)
    yb = whtmix.module_forward_separable(xd, wid, gtd, gcd, wod)
    poison(B, N, C, dtype, dev, True)
    gotb = whtmix.module_backward_separable(xd, wid, gtd, gcd, wod, dyd)
    torch.cuda.synchronize(dev)
    block = {"f32": 1e-5, "bf16": 4e-3}[dtype]
    checks = [("y", y, orc.whtmix_separable(x, gt, gc), DERIVED[dtype]),
              ("block y", yb, orc.whtmix_module_separable(x, wi, gt, gc, wo), block)]
    checks += zip(["dx", "dgt", "dgc"], got, orc.whtmix_grad_separable(x, dy, gt, gc),
                  [DERIVED[dtype], 1e-5, 1e-5])
    checks += zip(["block dx", "dw_in", "dw_out", "block dgt", "block dgc"], gotb,
                  orc.whtmix_module_grad_separable(x, wi, gt, gc, wo, dy), [block] + [1e-5] * 4)
    for name, t, ref, tol in checks:
        err = errors(to_host(t), ref)[0]
        assert err <= tol, (name, err)     # NaN fails too


@pytest.mark.parametrize("shape", [(1, 600, 256), (2, 1300, 256)],
                         ids=lambda s: "x".join(map(str, s)))
def test_padded_block_pair_tiles_left_out(shape, dev, orc):
    """The bf16 block with C = 256 on 2^16 outer tiles, the last of them wholly padded."""
    import torch

    B, N, C = shape
    P = whtmix.padded_tokens(N)
    x, _ = workloads.draw(B, N, C, "bf16", seed=720 + N)
    _, g = workloads.draw(1, P, C, "f32", seed=721 + N)
    wi, wo = workloads.draw_weights(C, "bf16", seed=722 + N)
    assert whtmix.plan_describe(B, N, C, "bf16")["module_outer_bits"] == 16
    say(f"padding pair-tile block {shape} bf16")
    xd, wid, wod = (to_device(t, "bf16", dev) for t in (x, wi, wo))
    gd = to_device(g, "f32", dev)
    poison(B, N, C, "bf16", dev, True)
    y = whtmix.module_forward(xd, wid, gd, wod)
    torch.cuda.synchronize(dev)
    assert errors(to_host(y), orc.whtmix_module(x, wi, g, wo))[0] <= 4e-3
