"""Which tile a folded product takes, at the lines of the rules: FP32 rows that
are not whole 16-byte pieces (odd channel counts at even orders, 45 entries a
channel), around a tile's rows and its batch, up to and above the reduction from
which they are treated like the others; the BF16 tiles for few rows and for wide
outputs; the voxel slices of the weight gradients.
"""
import numpy as np
import pytest
import torch

import datagen as dg
import paper_1808_01517_amd as dl

from parity_util import check

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _products(C, O, voxels, prec, store):
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(90), 8, 8, (8, 8), np.deg2rad(30), 0.006)
    W, b = dg.lsc_weights(8, 0, C, O, plan.T)
    W, b = (torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(DEV) for x in (W, b))
    gen = torch.Generator(device=DEV).manual_seed(8)
    a = torch.randn(voxels, C, plan.K_in, device=DEV, generator=gen)
    g = torch.randn(voxels, O, plan.K_out, device=DEV, generator=gen)
    if store == "half":
        a, g = a.bfloat16(), g.bfloat16()
    _, Bnb, Pm = (torch.from_numpy(np.asarray(t)).double() for t in plan.tables())
    Q = torch.einsum("ki,itj->tkj", Pm, Bnb.reshape(plan.m, plan.T, plan.K_in))
    T = torch.einsum("oct,tkj->okcj", W.double().cpu(), Q).reshape(O * plan.K_out, C * plan.K_in).to(DEV)
    bias = (b.double()[:, None] * Pm.sum(1).to(DEV)).reshape(-1)
    flat = a.reshape(voxels, -1)

    out = dl.lsc_fwd(plan, a, W, b, relu=True, precision=prec, out_dtype=a.dtype)
    check("out", out.float().reshape(voxels, -1), (flat.double() @ T.t() + bias).clamp(min=0.0), prec)
    ref = g.reshape(voxels, -1).double() @ T
    for relu_in in (False, True):
        da, _, _ = dl.lsc_bwd(plan, a, W, g, need_weight_grad=False, need_bias_grad=False, relu_in=relu_in,
                              precision=prec)
        check("da", da.float().reshape(voxels, -1), ref * (flat > 0) if relu_in else ref, prec)


# 45 onto 360 and back (64 x 48, 128 x 48 and 64 x 144 by batch), 1215 and 1305
# onto 180
@pytest.mark.parametrize("case,voxels",
                         [((1, 8), v) for v in (1, 63, 65, 4097, 8191, 16385, 40001)] +
                         [((27, 4), v) for v in (65, 8191, 16385)] + [((29, 4), v) for v in (65, 8191, 16385)])
def test_rows_of_pieces(case, voxels):
    _products(*case, voxels, "fp32", "fp32")
    _products(*case[::-1], voxels, "fp32", "fp32")


# BF16: onto 2880 columns the small tiles take up to 96 tiles of 128 x 144 (512
# rows), and the wide ones from 512 on, of bfloat16 rows only; onto 360 (three
# column tiles) the small ones take up to 4 096 rows
@pytest.mark.parametrize("store", ["fp32", "half"])
@pytest.mark.parametrize("case,voxels", [((8, 64), v) for v in (511, 512, 513, 4353, 4609)] +
                         [((64, 8), v) for v in (4095, 4096, 4097)])
def test_bf16_lines(case, voxels, store):
    _products(*case, voxels, "bf16", store)


# slices of 128 voxels up to a block for every compute unit, of 512 beyond: two
# column tiles of 144 by one to three row tiles here
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("case,voxels", [((4, 5), v) for v in (1, 127, 128, 255, 256, 257, 2000, 8191, 70001)])
def test_gradient_slices(case, voxels, masked, prec):
    C, O = case
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(90), 8, 8, (8, 8), np.deg2rad(30), 0.006)
    W = torch.from_numpy(np.ascontiguousarray(dg.lsc_weights(9, 0, C, O, plan.T)[0], dtype=np.float32)).to(DEV)
    gen = torch.Generator(device=DEV).manual_seed(9)
    a = torch.randn(voxels, C, plan.K_in, device=DEV, generator=gen)
    g, y = (torch.randn(voxels, O, plan.K_out, device=DEV, generator=gen) for _ in range(2))
    _, Bnb, Pm = (torch.from_numpy(np.asarray(t)).double().to(DEV) for t in plan.tables())
    Q = torch.einsum("ki,itj->tkj", Pm, Bnb.reshape(plan.m, plan.T, plan.K_in))
    gm = (g * (y > 0) if masked else g).double()
    dT = (gm.reshape(voxels, -1).t() @ a.reshape(voxels, -1).double()).reshape(O, plan.K_out, C, plan.K_in)
    kw = {"a_out": y, "relu": True} if masked else {}
    _, dW, db = dl.lsc_bwd(plan, a, W, g, need_input_grad=False, precision=prec, **kw)
    check("dW", dW, torch.einsum("okcj,tkj->oct", dT, Q), prec, kind="sum")
    check("db", db, (gm.sum(0) * Pm.sum(1)).sum(1), prec, kind="sum")
