"""FP32 folded layers on values that three bfloat16 parts do not hold
(csrc/parts.h): weights whose folded entries are infinite, NaN or above
bfloat16's range, through every core (short reductions, streaming tiles,
images), with float32's results.
"""
import numpy as np
import pytest
import torch

import datagen as dg
import paper_1808_01517_amd as dl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


def same_specials(out, ref, rtol):
    out = out.double().cpu().numpy().reshape(ref.shape)
    assert np.array_equal(np.isnan(out), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(out[inf], ref[inf])
    fin = np.isfinite(ref)
    np.testing.assert_allclose(out[fin], ref[fin], rtol=rtol, atol=0)


@pytest.mark.parametrize("layer", [(3, 2, 70), (135, 32, 300), (32, 135, 33), (300 - 44, 5, 130), (1, 1, 1)])
def test_weights_beyond_the_parts(layer):
    # order 0: the folded matrix is q W[o][c][0] for a weight with one tap, so
    # its entries can be put anywhere; products of the large ones are finite
    C, O, V = layer
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(12), 0, 0, (6,), np.deg2rad(30), 0.006)
    _, Bnb, Pm = plan.tables()
    q = np.float32((Pm @ Bnb.reshape(plan.m, plan.T, 1)[:, 0])[0, 0])
    rng = np.random.default_rng(21)
    W = np.zeros((O, C, plan.T), np.float32)
    W[:, :, 0] = rng.standard_normal((O, C))
    special = [np.inf, -np.inf, np.nan, np.float32(3.4e38) / q, np.float32(-3.4e38) / q]
    for i, x in enumerate(special):
        W[i % O, (2 * i) % C, 0] = x
    with np.errstate(over="ignore"):
        T = (W[:, :, 0] * q).astype(np.float64)
    big = np.isfinite(T) & (np.abs(T) > 3.39e38)
    assert big.any() or layer == (1, 1, 1)
    a = (0.25 * rng.uniform(0.5, 1.0, (V, C)) * rng.choice([-1.0, 1.0], (V, C))).astype(np.float32)
    g = (0.25 * rng.uniform(0.5, 1.0, (V, O)) * rng.choice([-1.0, 1.0], (V, O))).astype(np.float32)
    a[0, 0] = 0.0
    with np.errstate(invalid="ignore"):
        ref = np.stack([(x.astype(np.float64) * T).sum(1) for x in a])
        rda = np.stack([(x.astype(np.float64)[:, None] * T).sum(0) for x in g])
    # rows without special weights: float32 rounding of sums of up to 256 terms
    # that may cancel; the large ones dominate their sums
    for r in (ref, rda):
        small = np.isfinite(r) & (np.abs(r) < 1e30)
        r[small] = np.round(r[small], 3)

    def close(out, r):
        out = out.double().cpu().numpy().reshape(r.shape)
        small = np.isfinite(r) & (np.abs(r) < 1e30)
        assert np.abs(out[small] - r[small]).max(initial=0.0) <= 2e-3
        out[small] = r[small]
        same_specials(torch.from_numpy(out), r, 1e-6)

    ag, gg, Wg = cuda(a.reshape(V, C, 1)), cuda(g.reshape(V, O, 1)), cuda(W)
    close(dl.lsc_fwd(plan, ag, Wg, None), ref)
    da, _, _ = dl.lsc_bwd(plan, ag, Wg, gg, need_weight_grad=False, need_bias_grad=False)
    close(da, rda)
    ai, gi = cuda(a.T.reshape(1, C, V)), cuda(g.T.reshape(1, O, V))
    out, _ = dl.lsc_fwd_image(plan, ai, Wg)
    close(out[0].t(), ref)
    da, _, _ = dl.lsc_bwd_image(plan, ai, Wg, gi, need_weight_grad=False, need_bias_grad=False)
    close(da[0].t(), rda)
