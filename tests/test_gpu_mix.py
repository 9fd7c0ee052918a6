"""The resample form with the channels mixed before the resampling (FP32
layers for which that order takes fewer multiplications): the smallest and
ragged batches, several passes through a small workspace, equal channel
counts, the input-gradient mask, gradients left out.  Held to the FP64 oracle.
"""
import numpy as np
import pytest
import torch

import datagen as dg
import paper_1808_01517_amd as dl
from oracle import lsc as olsc

from parity_util import check

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


@pytest.mark.parametrize("case", [
    (32, 3, 8, 8, (8, 8), 90, 1), (32, 3, 8, 8, (8, 8), 90, 67), (9, 1, 4, 2, (6,), 30, 33),
    (16, 16, 4, 4, (6, 6), 60, 130), (5, 4, 2, 4, (3, 4, 5), 45, 257), (4, 3, 6, 6, (8,), 28, 50),
])
@pytest.mark.parametrize("relu_in", [False, True])
def test_mixed_order_matches_oracle(case, relu_in):
    C, O, L_in, L_out, ks, m, V = case
    g = dg.fibonacci_hemisphere(m)
    oplan = olsc.LSCPlan(g, L_in, L_out, ks, np.deg2rad(30), 0.006)
    plan = dl.LSCPlan(g, L_in, L_out, ks, np.deg2rad(30), 0.006)
    W, b = (x.astype(np.float32).astype(np.float64) for x in dg.lsc_weights(8, 0, C, O, plan.T))
    rng = np.random.default_rng(8)
    a = rng.standard_normal((V, C, plan.K_in)).astype(np.float32).astype(np.float64)
    da_out = rng.standard_normal((V, O, plan.K_out)).astype(np.float32).astype(np.float64)
    ref, z = olsc.lsc_forward(oplan, a, W, b, True)
    da_ref, dW_ref, db_ref = olsc.lsc_backward(oplan, a, W, z, da_out, False)
    if relu_in:
        da_ref = da_ref * (a > 0)
    ws = dl.Workspace(dl.lsc_workspace_bytes(plan, C, O, 64, "fp32", "resample"), DEV)  # 64 voxels a pass
    for w in (None, ws):
        check("out", dl.lsc_fwd(plan, cuda(a), cuda(W), cuda(b), relu=True, form="resample", workspace=w), ref, "fp32")
        out = dl.lsc_fwd(plan, cuda(a), cuda(W), None, form="resample", workspace=w)
        check("out without bias", out, olsc.lsc_forward(oplan, a, W, 0 * b, False)[0], "fp32")
        da, dW, db = dl.lsc_bwd(plan, cuda(a), cuda(W), cuda(da_out), form="resample", relu_in=relu_in, workspace=w)
        check("da", da, da_ref, "fp32")
        check("dW", dW, dW_ref, "fp32", kind="sum")
        check("db", db, db_ref, "fp32", kind="sum")
        da, dW, db = dl.lsc_bwd(plan, cuda(a), cuda(W), cuda(da_out), form="resample", relu_in=relu_in, workspace=w,
                                need_weight_grad=False, need_bias_grad=False)
        assert dW is None and db is None
        check("da alone", da, da_ref, "fp32")
        da, dW, db = dl.lsc_bwd(plan, cuda(a), cuda(W), cuda(da_out), form="resample", workspace=w,
                                need_input_grad=False, need_bias_grad=False)
        assert da is None and db is None
        check("dW alone", dW, dW_ref, "fp32", kind="sum")


@pytest.mark.parametrize("case", [(32, 3), (16, 16), (9, 1)])
def test_mixed_order_is_as_close_as_the_papers(case):
    # With u = 2^-24 / sqrt(3) the rounding of one sum, a running sum of n equal
    # terms, four to a rounding, is off by u sqrt(n / 8).  T K = 765 of them in
    # pieces of 128: 1.5e-7 (in one piece 3.4e-7); with the sum over the channels
    # and the refit's 90 2.0e-7 (3.6e-7).  The bound is between; the paper's order,
    # with sums over 45, C T and 90 entries, measured 2.2e-7 to 3.4e-7.
    C, O = case
    g = dg.fibonacci_hemisphere(90)
    plan = dl.LSCPlan(g, 8, 8, (8, 8), np.deg2rad(30), 0.006)
    oplan = olsc.LSCPlan(g, 8, 8, (8, 8), np.deg2rad(30), 0.006)
    W, b = (x.astype(np.float32).astype(np.float64) for x in dg.lsc_weights(9, 0, C, O, plan.T))
    a = np.random.default_rng(9).standard_normal((300, C, plan.K_in)).astype(np.float32).astype(np.float64)
    ref = olsc.lsc_forward(oplan, a, W, b, False)[0]
    out = dl.lsc_fwd(plan, cuda(a), cuda(W), cuda(b), form="resample").double().cpu().numpy()
    assert np.linalg.norm(out - ref) <= 2.8e-7 * np.linalg.norm(ref)


def test_rows_beyond_32_bits():
    # 2^31 rows (voxel, output channel) in one workspace: the call takes them in passes
    C, O = 128, 256
    V = 2 ** 31 // O + 5
    g = dg.fibonacci_hemisphere(3)
    plan = dl.LSCPlan(g, 0, 0, (2,), np.deg2rad(30), 0.006)
    W, b = (x.astype(np.float32).astype(np.float64) for x in dg.lsc_weights(10, 0, C, O, plan.T))
    gen = torch.Generator(device=DEV).manual_seed(10)
    a = torch.randn(V, C, 1, device=DEV, generator=gen)
    ws = dl.Workspace(dl.lsc_workspace_bytes(plan, C, O, V, "fp32", "resample"), DEV)
    out = dl.lsc_fwd(plan, a, cuda(W), cuda(b), form="resample", workspace=ws)
    rows = [0, 1, V // 2, 2 ** 30 // O - 1, 2 ** 30 // O, V - 2, V - 1]
    oplan = olsc.LSCPlan(g, 0, 0, (2,), np.deg2rad(30), 0.006)
    ref = olsc.lsc_forward(oplan, a[rows].double().cpu().numpy(), W, b, False)[0]
    check("out", out[rows], ref, "fp32")


# the forward's line, in voxels a pass: 13 000 K <= V (C m - O K), just below, at
# and above it, and a last pass of any size
@pytest.mark.parametrize("case,line", [((32, 3, 8, 8, (8, 8), 90), 214), ((16, 16, 4, 4, (6, 6), 60), 271),
                                       ((9, 1, 4, 2, (6,), 30), 765), ((5, 4, 2, 4, (3, 4, 5), 45), 389)])
def test_mixed_forward_from_its_line_on(case, line):
    C, O, L_in, L_out, ks, m = case
    g = dg.fibonacci_hemisphere(m)
    oplan = olsc.LSCPlan(g, L_in, L_out, ks, np.deg2rad(30), 0.006)
    plan = dl.LSCPlan(g, L_in, L_out, ks, np.deg2rad(30), 0.006)
    assert (line - 1) * (C * m - O * plan.K_in) < 13000 * plan.K_in <= line * (C * m - O * plan.K_in)
    W, b = (x.astype(np.float32).astype(np.float64) for x in dg.lsc_weights(11, 0, C, O, plan.T))
    V = 2 * line + 65
    a = np.random.default_rng(11).standard_normal((V, C, plan.K_in)).astype(np.float32).astype(np.float64)
    ref = olsc.lsc_forward(oplan, a, W, b, True)[0]
    ag, Wg, bg = cuda(a), cuda(W), cuda(b)
    for n in (line - 1, line, line + 1, V):
        check("out", dl.lsc_fwd(plan, ag[:n], Wg, bg, relu=True, form="resample"), ref[:n], "fp32")
    for per in (line - 1, line, line + 63):
        ws = dl.Workspace(dl.lsc_workspace_bytes(plan, C, O, per, "fp32", "resample"), DEV)
        check("passes", dl.lsc_fwd(plan, ag, Wg, bg, relu=True, form="resample", workspace=ws), ref, "fp32")
