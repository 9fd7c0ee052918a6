"""The fold of the kernel tensor and its adjoint (csrc/fold.hip) where their
blocks end: taps beyond one group of 16 and beyond the 32 held at a time, more
than 2048 coefficient pairs, channel counts that leave a ragged last block,
and few and many voxel slices of the weight gradient.  Held to the FP64
oracle through the layer, with the parity tests' tolerances.
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
    (1, 1, 0, 2, (4,), 12, 5),        # one pair, one input coefficient
    (3, 3, 4, 4, (15,), 30, 70),      # 16 taps: one whole group
    (2, 5, 4, 6, (8, 24), 45, 70),    # 33 taps: a second pass over the taps
    (2, 3, 10, 10, (8, 8), 90, 40),   # 66 x 66 pairs: three gradient chunks
    (5, 128, 2, 2, (6, 6), 12, 90),   # four channels per block, the last block ragged
    (2, 3, 4, 4, (6, 6), 30, 1100),   # two voxel slices
    (2, 3, 4, 4, (6, 6), 30, 2100),   # four: summed by a pass of their own
])
def test_fold_and_unfold_edges(case):
    C, O, L_in, L_out, ks, m, V = case
    g = dg.fibonacci_hemisphere(m)
    oplan = olsc.LSCPlan(g, L_in, L_out, ks, np.deg2rad(30), 0.006)
    plan = dl.LSCPlan(g, L_in, L_out, ks, np.deg2rad(30), 0.006)
    W, b = dg.lsc_weights(7, 0, C, O, plan.T)
    W, b = (x.astype(np.float32).astype(np.float64) for x in (W, b))
    rng = np.random.default_rng(7)
    a = rng.standard_normal((V, C, plan.K_in)).astype(np.float32).astype(np.float64)
    g_out = rng.standard_normal((V, O, plan.K_out)).astype(np.float32).astype(np.float64)
    ref, z = olsc.lsc_forward(oplan, a, W, b, False)
    da_ref, dW_ref, db_ref = olsc.lsc_backward(oplan, a, W, z, g_out, False)
    check("out", dl.lsc_fwd(plan, cuda(a), cuda(W), cuda(b)), ref, "fp32")
    da, dW, db = dl.lsc_bwd(plan, cuda(a), cuda(W), cuda(g_out))
    check("da", da, da_ref, "fp32")
    check("dW", dW, dW_ref, "fp32", kind="sum")
    check("db", db, db_ref, "fp32", kind="sum")
