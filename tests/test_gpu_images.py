"""The layers on 5-D images (csrc/image.hip, csrc/tile.hip) against the
voxel-major calls of the same layers on the permuted data: sizes around the
tiles and the 16-byte runs, every transform, the ReLU bits, memory orders of
the input, and in-place changes after the forward.  FP32 differs in the order
of its sums only; BF16 forwards are the same bits.
"""
import numpy as np
import pytest
import torch

import datagen as dg
import paper_1808_01517_amd as dl
from paper_1808_01517_amd.layers import LocalSphericalConvolution, SH2Signal, Signal2SH

from parity_util import TOL, rel

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(1, 1, 1, 1), (2, 1, 1, 3), (1, 3, 3, 7), (3, 4, 4, 4), (1, 5, 5, 5), (2, 1, 1, 129), (1, 1, 15, 17),
          (1, 8, 32, 9)]


def flat(x):
    return x.permute(0, 2, 3, 4, 1).reshape(-1, x.shape[1]).contiguous()


def image(v, like):
    B, _, H, W, D = like.shape
    return v.reshape(B, H, W, D, -1).permute(0, 4, 1, 2, 3).contiguous()


def rand(gen, *s):
    return torch.randn(*s, device=DEV, generator=gen)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("table", [((30,), 4), ((45, 90, 17), 4), ((90, 90, 90), 8), ((96, 128), 12)])
def test_sh_transforms(table, prec):
    dirs, L = table
    rng = np.random.default_rng(1)
    g = np.concatenate([dg.fibonacci_hemisphere(n) + rng.uniform(-0.01, 0.01, (n, 3)) for n in dirs])
    b = np.concatenate([np.full(n, 1000.0 * (k + 1)) for k, n in enumerate(dirs)])
    s2sh, sh2s = Signal2SH(L, g, b, precision=prec), SH2Signal(L, g, b, precision=prec)
    gen = torch.Generator(device=DEV).manual_seed(2)
    n, k = s2sh.plan.n_dw, s2sh.plan.n_shells * s2sh.plan.K
    for B, H, W, D in SHAPES[::2] if L > 4 else SHAPES:
        x, c = rand(gen, B, n, H, W, D).requires_grad_(), rand(gen, B, k, H, W, D).requires_grad_()
        for mod, inp, other, fwd, bwd in ((s2sh, x, c, dl.signal2sh_fwd, dl.signal2sh_bwd),
                                          (sh2s, c, x, dl.sh2signal_fwd, dl.sh2signal_bwd)):
            out = mod(inp)
            assert out.is_contiguous() and out.shape == other.shape
            grad, = torch.autograd.grad(out, inp, other.detach())
            shape = (-1, mod.plan.n_shells, mod.plan.K)
            vin, vg = flat(inp.detach()), flat(other.detach())
            ref = fwd(mod.plan, vin if mod is s2sh else vin.reshape(shape), precision=prec)
            rgr = bwd(mod.plan, vg.reshape(shape) if mod is s2sh else vg, precision=prec)
            ref, rgr = image(ref.reshape(ref.shape[0], -1), out), image(rgr.reshape(rgr.shape[0], -1), grad)
            if prec == "bf16":
                assert torch.equal(out, ref) and torch.equal(grad, rgr)
            else:
                assert rel(out, ref) <= TOL[prec] and rel(grad, rgr) <= TOL[prec]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("layer", [(1, 8, 4), (3, 32, 8), (32, 3, 8), (2, 3, 2), (1, 1, 0)])
def test_lsc(layer, relu, prec):
    C, O, L = layer
    conv = LocalSphericalConvolution(C, O, dg.fibonacci_hemisphere(90), L, L, (8, 8), np.deg2rad(30), relu=relu,
                                     precision=prec).to(DEV)
    gen = torch.Generator(device=DEV).manual_seed(3)
    K = conv.plan.K_in
    for B, H, W, D in SHAPES:
        a = rand(gen, B, C * K, H, W, D).requires_grad_()
        g = rand(gen, B, O * K, H, W, D)
        out = conv(a)
        assert out.is_contiguous()
        va = flat(a.detach()).reshape(-1, C, K)
        Wt, bias = conv.sconv.weight.detach(), conv.sconv.bias.detach()
        ref = dl.lsc_fwd(conv.plan, va, Wt, bias, relu=relu, precision=prec)
        if prec == "bf16":
            assert torch.equal(out, image(ref.reshape(ref.shape[0], -1), out))
        else:
            assert rel(out, image(ref.reshape(ref.shape[0], -1), out)) <= TOL[prec]
        vout = flat(out.detach()).reshape(-1, O, K)  # the same ReLU pattern on both sides
        grads = torch.autograd.grad(out, [a, conv.sconv.weight, conv.sconv.bias], g)
        da, dW, db = dl.lsc_bwd(conv.plan, va, Wt, flat(g).reshape(-1, O, K), a_out=vout, relu=relu, precision=prec)
        tol = TOL[prec] if prec == "fp32" else 1e-5  # BF16 rounds the same operands: the sums' order differs only
        for got, want in zip(grads, (image(da.reshape(da.shape[0], -1), a), dW.view_as(Wt), db)):
            assert rel(got, want) <= tol


def test_memory_orders_and_late_changes():
    conv = LocalSphericalConvolution(2, 3, dg.fibonacci_hemisphere(30), 4, 4, (6, 6), np.deg2rad(30), relu=True).to(DEV)
    gen = torch.Generator(device=DEV).manual_seed(4)
    a = rand(gen, 2, 30, 3, 5, 7)
    g = rand(gen, 2, 45, 3, 5, 7)
    params = [conv.sconv.weight, conv.sconv.bias]
    want = conv(a)
    ref = torch.autograd.grad(want, params, g)
    for view in (a.permute(0, 2, 3, 4, 1).contiguous().permute(0, 4, 1, 2, 3),      # voxel-major memory
                 a.transpose(2, 4).contiguous().transpose(2, 4),                    # neither order
                 torch.cat([a, a], 1)[:, :30], a[:, :, :, :, torch.arange(7, device=DEV)]):
        out = conv(view)
        assert out.is_contiguous() and rel(out, want) <= TOL["fp32"]
        for x, y in zip(torch.autograd.grad(out, params, g), ref):
            assert rel(x, y) <= TOL["fp32"]
    # the caller may change its input and the output before the backward
    b = a.clone()
    out = conv(b)
    b.zero_()
    with torch.no_grad():
        out.zero_()
    for x, y in zip(torch.autograd.grad(out, params, g), ref):
        assert torch.equal(x, y)
    with pytest.raises(ValueError):
        conv(a[:, :29])


def test_more_images_than_one_launch_takes():
    conv = LocalSphericalConvolution(1, 2, dg.fibonacci_hemisphere(30), 2, 2, (6,), np.deg2rad(30)).to(DEV)
    gen = torch.Generator(device=DEV).manual_seed(5)
    a = rand(gen, 129, 6, 2, 1, 3)
    out = conv(a)
    ref = torch.cat([conv(a[:100]), conv(a[100:])])
    assert rel(out, ref) <= TOL["fp32"]
    g = rand(gen, *out.shape)
    dW, = torch.autograd.grad(out, [conv.sconv.weight], g)
    r = [torch.autograd.grad(conv(a[s]), [conv.sconv.weight], g[s])[0] for s in (slice(0, 100), slice(100, 129))]
    assert rel(dW, r[0] + r[1]) <= TOL["fp32"]
