"""The tiles of the streaming table products (csrc/stream.hip), each at rows
just before, at and after a tile of its own, with reductions that end inside a
stage: every FP32 tile that the batch size chooses between, and the BF16 tiles
for few rows, for wide outputs and for the rest.
"""
import numpy as np
import pytest
import torch

import datagen as dg
import paper_1808_01517_amd as dl

from parity_util import check

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# batches onto 2880 columns by the FP32 tile they take: 64 x 48 (ring of four),
# 64 x 144, 256 x 96, 128 x 48, 256 x 144
FP32_ROWS = [1, 63, 64, 65, 513, 575, 577, 1601, 1793, 2049, 2175, 2433, 2561]
# 64 x 48 (ring of eight) below 128 tiles of 128 x 144, then 128 x 144, then
# 256 x 96 without a mask from 512 tiles on
BF16_ROWS = [1, 63, 64, 65, 768, 769, 897, 4352, 4353, 4609]


@pytest.mark.parametrize("prec,store,voxels",
                         [("fp32", "fp32", v) for v in FP32_ROWS] + [("bf16", "fp32", v) for v in BF16_ROWS[1::2]] +
                         [("bf16", "half", v) for v in BF16_ROWS])
@pytest.mark.parametrize("flip", [False, True])
def test_tiles(flip, prec, store, voxels):
    # 8 x 45 = 360 (eleven stages and a quarter) onto 64 x 45 = 2880, and back
    C, O = (64, 8) if flip else (8, 64)
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(90), 8, 8, (8, 8), np.deg2rad(30), 0.006)
    W, b = dg.lsc_weights(6, 0, C, O, plan.T)
    W, b = (torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(DEV) for x in (W, b))
    gen = torch.Generator(device=DEV).manual_seed(6)
    a = torch.randn(voxels, C, plan.K_in, device=DEV, generator=gen)
    g = torch.randn(voxels, O, plan.K_out, device=DEV, generator=gen)
    if store == "half":
        a, g = a.bfloat16(), g.bfloat16()
    _, Bnb, Pm = (torch.from_numpy(np.asarray(t)).double() for t in plan.tables())
    Q = torch.einsum("ki,itj->tkj", Pm, Bnb.reshape(plan.m, plan.T, plan.K_in))
    T = torch.einsum("oct,tkj->okcj", W.double().cpu(), Q).reshape(O * plan.K_out, C * plan.K_in).to(DEV)
    bias = (b.double()[:, None] * Pm.sum(1).to(DEV)).reshape(-1)

    pre = a.reshape(voxels, -1).double() @ T.t() + bias
    kind = a.dtype
    out = dl.lsc_fwd(plan, a, W, b, precision=prec, out_dtype=kind)
    check("out", out.float().reshape(voxels, -1), pre, prec)
    out = dl.lsc_fwd(plan, a, W, b, relu=True, precision=prec, out_dtype=kind)
    check("relu", out.float().reshape(voxels, -1), pre.clamp(min=0.0), prec)

    ref = g.reshape(voxels, -1).double() @ T
    for relu_in in (False, True):
        da, _, _ = dl.lsc_bwd(plan, a, W, g, need_weight_grad=False, need_bias_grad=False, relu_in=relu_in,
                              precision=prec)
        check("da", da.float().reshape(voxels, -1), ref * (a.reshape(voxels, -1) > 0) if relu_in else ref, prec)
