"""Image layers with some gradients left out: a layer whose parameters are
frozen keeps nothing of its input, which may change in place before the
backward; each gradient alone is the one of the whole backward.
"""
import numpy as np
import pytest
import torch

import datagen as dg
import paper_1808_01517_amd as dl
from paper_1808_01517_amd.layers import LocalSphericalConvolution

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("relu", [False, True])
def test_frozen_layers(relu, prec):
    conv = LocalSphericalConvolution(2, 3, dg.fibonacci_hemisphere(30), 4, 4, (6, 6), np.deg2rad(30), relu=relu,
                                     precision=prec).to(DEV)
    gen = torch.Generator(device=DEV).manual_seed(14)
    x = torch.randn(2, 30, 3, 5, 7, device=DEV, generator=gen, requires_grad=True)
    g = torch.randn(2, 45, 3, 5, 7, device=DEV, generator=gen)
    W, b = conv.sconv.weight, conv.sconv.bias
    want = torch.autograd.grad(conv(x * 1), [x, W, b], g)
    for grads in ((False, False), (True, False), (False, True)):
        W.requires_grad_(grads[0])
        b.requires_grad_(grads[1])
        h = x * 1
        out = conv(h)
        saved = [t for t in out.grad_fn.saved_tensors if t is not None and t.shape == h.shape]
        assert len(saved) == any(grads) and all(t.data_ptr() != h.data_ptr() for t in saved)
        with torch.no_grad():
            h.zero_()
        got = torch.autograd.grad(out, [x] + [p for p, n in zip((W, b), grads) if n], g)
        for y, z in zip(got, [want[0]] + [w for w, n in zip(want[1:], grads) if n]):
            assert torch.equal(y, z)


def test_no_input_without_weight_gradients():
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(30), 2, 2, (6,), np.deg2rad(30), 0.006)
    gen = torch.Generator(device=DEV).manual_seed(15)
    a, g = (torch.randn(1, n * plan.K_in, 40, device=DEV, generator=gen) for n in (2, 3))
    W = torch.randn(3, 2, plan.T, device=DEV, generator=gen)
    da = dl.lsc_bwd_image(plan, None, W, g, need_weight_grad=False, need_bias_grad=False)[0]
    assert torch.equal(da, dl.lsc_bwd_image(plan, a, W, g)[0])
    for kw in ({"need_weight_grad": False}, {"need_bias_grad": False}):
        with pytest.raises(ValueError):
            dl.lsc_bwd_image(plan, None, W, g, **kw)
    for bad in (a[:, :-1], a[:, :, 1:]):
        with pytest.raises(ValueError):
            dl.lsc_bwd_image(plan, bad.contiguous(), W, g)
    for bad in (g[:, 1:].contiguous(), W):
        with pytest.raises(ValueError):
            dl.lsc_bwd_image(plan, a, W, bad)
    with pytest.raises(ValueError):
        dl.lsc_bwd_image(plan, a, W, g, torch.zeros(1, 3, 3, dtype=torch.int16, device=DEV))


def test_voxel_axes_of_the_backward():
    # any number of voxel axes, none for one voxel; the gradient and the input
    # need not have the same ones
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(30), 2, 2, (6,), np.deg2rad(30), 0.006)
    gen = torch.Generator(device=DEV).manual_seed(16)
    W = torch.randn(3, 2, plan.T, device=DEV, generator=gen)
    for axes, other in (((1,), ()), ((30,), (2, 3, 5)), ((2, 3, 5), (6, 5))):
        a, g = (torch.randn(2, n * plan.K_in, *axes, device=DEV, generator=gen) for n in (2, 3))
        _, bits = dl.lsc_fwd_image(plan, a, W, relu=True, need_bits=True)
        want = dl.lsc_bwd_image(plan, a, W, g, bits)
        flat = bits.view(torch.uint16).flatten()
        for a2, g2, b2 in ((a.view(2, -1, *other), g, bits), (a, g.view(2, -1, *other), flat)):
            got = dl.lsc_bwd_image(plan, a2, W, g2, b2)
            assert got[0].shape == a2.shape and torch.equal(got[0].flatten(), want[0].flatten())
            assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
