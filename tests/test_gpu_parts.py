"""FP32 on the bfloat16 matrix cores (csrc/parts.h) and the register-staged
weight gradient (csrc/tile.hip) where they can go wrong: infinities, NaN and
values beyond bfloat16's range, rows shorter than a 16-byte run, matrices that
end just before, at and after a tile, voxel counts around a stage of 32.
"""
import numpy as np
import pytest
import torch

import datagen as dg
import paper_1808_01517_amd as dl

from parity_util import check

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


def _plan(L_in, L_out, m=30, ks=(6,)):
    return dl.LSCPlan(dg.fibonacci_hemisphere(m), L_in, L_out, ks, np.deg2rad(30), 0.006)


def _folded(plan, W):
    """(T [O*K_out][C*K_in], Q) in float64 from the plan's own tables."""
    _, Bnb, Pm = plan.tables()
    Q = np.einsum("ki,itj->tkj", Pm, Bnb.reshape(plan.m, plan.T, plan.K_in))
    O, C, _ = W.shape
    T = np.einsum("oct,tkj->okcj", W, Q).reshape(O * plan.K_out, C * plan.K_in)
    return T, Q


def _same_specials(out, ref):
    out = out.double().cpu().numpy().reshape(ref.shape)
    assert np.array_equal(np.isnan(out), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(out[inf], ref[inf])
    fin = np.isfinite(ref)
    assert np.isfinite(out[fin]).all()
    return out, fin


@pytest.mark.parametrize("shape", [(3, 32, 8, 203), (32, 3, 8, 70), (8, 16, 4, 300), (9, 3, 4, 40)])
def test_specials_follow_float32(shape):
    # K = 135 (short-reduction kernel), 1440, 120 and 135 again with N = 45;
    # the float32 product of a 2^127-sized value with entries below 1 is finite
    C, O, L, V = shape
    plan = _plan(L, L, m=90 if L == 8 else 30, ks=(8, 8))
    W = dg.lsc_weights(3, 0, C, O, plan.T)[0].astype(np.float32).astype(np.float64)
    rng = np.random.default_rng(3)
    a = rng.standard_normal((V, C * plan.K_in)).astype(np.float32)
    a[1, 2], a[5, 0], a[7, 7], a[9, 3], a[9, 4] = np.inf, -np.inf, np.nan, np.inf, -np.inf
    a[V - 1, 1] = 3.4e38
    T, Q = _folded(plan, W)
    T = T.astype(np.float32).astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = np.stack([(a[v].astype(np.float64) * T).sum(1) for v in range(V)])
    out = dl.lsc_fwd(plan, cuda(a.reshape(V, C, -1)), cuda(W), None)
    got, fin = _same_specials(out, ref)
    np.testing.assert_allclose(got[fin], ref[fin], rtol=1e-3, atol=1e-4)
    # the weight gradient of that input: every entry an infinite or NaN
    # voxel reaches is infinite or NaN as float32 has it, the others finite
    g = rng.standard_normal((V, O * plan.K_out)).astype(np.float32)
    g[11, 5] = np.inf
    b = np.where(np.isfinite(a), a, 0.0)
    b[V - 1, 1] = 1.0
    _, dW, db = dl.lsc_bwd(plan, cuda(b.reshape(V, C, -1)), cuda(W), cuda(g.reshape(V, O, -1)))
    o_bad = 5 // plan.K_out
    keep = np.arange(O) != o_bad
    assert np.isfinite(dW.cpu().numpy()[keep]).all() and not np.isfinite(dW.cpu().numpy()[o_bad]).any()
    assert np.isinf(db.cpu().numpy()[o_bad]) and np.isfinite(db.cpu().numpy()[keep]).all()


@pytest.mark.parametrize("store", ["fp32", "bf16", "half"])
@pytest.mark.parametrize("case", [
    (1, 1, 0, 0, 1), (1, 3, 0, 0, 33),           # rows of 1 and 3 entries: no 16-byte runs
    (1, 1, 0, 2, 31), (4, 5, 0, 0, 32),
    (142, 127, 0, 0, 63), (143, 128, 0, 0, 64), (144, 129, 0, 0, 65),  # around the 128 x 144 tile
    (128, 143, 0, 0, 700), (8, 144, 0, 0, 1100), (136, 8, 0, 0, 1024),
])
def test_weight_gradient_edges(case, store):
    C, O, L_in, L_out, V = case
    if store == "half" and (C % 8 or O % 8):
        pytest.skip("bfloat16 rows need multiples of 8 entries")
    prec = "fp32" if store == "fp32" else "bf16"
    plan = _plan(L_in, L_out)
    W = dg.lsc_weights(4, 0, C, O, plan.T)[0]
    rng = np.random.default_rng(4)
    a = rng.standard_normal((V, C, plan.K_in)).astype(np.float32)
    g = rng.standard_normal((V, O, plan.K_out)).astype(np.float32)
    ag, gg = cuda(a), cuda(g)
    if store == "half":
        ag, gg = ag.bfloat16(), gg.bfloat16()
        a, g = ag.float().cpu().numpy(), gg.float().cpu().numpy()
    _, Q = _folded(plan, W.astype(np.float64))
    _, _, Pm = plan.tables()
    G = g.reshape(V, -1).astype(np.float64).T @ a.reshape(V, -1).astype(np.float64)
    dW_ref = np.einsum("okcj,tkj->oct", G.reshape(O, plan.K_out, C, plan.K_in), Q)
    db_ref = g.astype(np.float64).sum(0) @ Pm.sum(1)
    _, dW, db = dl.lsc_bwd(plan, ag, cuda(W), gg, need_input_grad=False, precision=prec)
    check("dW", dW, dW_ref, prec, kind="sum")
    check("db", db, db_ref, prec, kind="sum")
    if store == "fp32":  # masked by the layer's own output
        mask = rng.standard_normal(g.shape).astype(np.float32)
        gm = g * (mask > 0)
        G = gm.reshape(V, -1).astype(np.float64).T @ a.reshape(V, -1).astype(np.float64)
        _, dW, db = dl.lsc_bwd(plan, ag, cuda(W), gg, a_out=cuda(mask), relu=True, need_input_grad=False)
        check("dW masked", dW, np.einsum("okcj,tkj->oct", G.reshape(O, plan.K_out, C, plan.K_in), Q), prec, kind="sum")
        check("db masked", db, gm.astype(np.float64).sum(0) @ Pm.sum(1), prec, kind="sum")


@pytest.mark.parametrize("case", [(1, 8, 4), (3, 32, 4), (8, 3, 4)])
def test_long_sums_do_not_drift(case):
    # 131 072 voxels in slices of 1024 or more: 32 steps of 2^-24 each, at random,
    # are 3.4e-7 of a slice's sum; a cut always to one side grows with the steps
    C, O, L = case
    V = 131072
    plan = _plan(L, L)
    W = dg.lsc_weights(8, 0, C, O, plan.T)[0]
    gen = torch.Generator(device=DEV).manual_seed(8)
    a = torch.randn(V, C, plan.K_in, device=DEV, generator=gen)
    g = torch.randn(V, O, plan.K_out, device=DEV, generator=gen)
    _, Q = _folded(plan, W.astype(np.float64))
    G = (g.reshape(V, -1).double().t() @ a.reshape(V, -1).double()).cpu().numpy()
    ref = np.einsum("okcj,tkj->oct", G.reshape(O, plan.K_out, C, plan.K_in), Q)
    _, dW, _ = dl.lsc_bwd(plan, a, cuda(W), g, need_input_grad=False)
    err = np.linalg.norm(dW.double().cpu().numpy().reshape(ref.shape) - ref) / np.linalg.norm(ref)
    assert err <= 3.4e-7, err


@pytest.mark.parametrize("positive", [False, True])
@pytest.mark.parametrize("case", [(256, 3, 200), (256, 64, 300), (64, 256, 300)])
def test_longest_reductions(case, positive):
    # 256 channels of order 8, 11 520 entries: the float32 instruction's running
    # sum, four entries to a rounding of 2^-24 / sqrt(3), is off by sqrt(K / 8) of
    # them, 1.3e-6 (measured 1.9e-6); the part products are held to it, also
    # where every product is positive and the matrix unit's cuts add up
    C, O, V = case
    plan = _plan(8, 8, m=90, ks=(8, 8))
    W = dg.lsc_weights(11, 0, C, O, plan.T)[0].astype(np.float32).astype(np.float64)
    rng = np.random.default_rng(11)
    a = rng.standard_normal((V, C * plan.K_in)).astype(np.float32)
    g = rng.standard_normal((V, O * plan.K_out)).astype(np.float32)
    if positive:
        W, a, g = np.abs(W), np.abs(a), np.abs(g)
    T, _ = _folded(plan, W)
    T = torch.from_numpy(T).to(DEV)
    ag, gg, Wg = cuda(a.reshape(V, C, -1)), cuda(g.reshape(V, O, -1)), cuda(W)
    out = dl.lsc_fwd(plan, ag, Wg, None).reshape(V, -1).double()
    da = dl.lsc_bwd(plan, ag, Wg, gg, need_weight_grad=False, need_bias_grad=False)[0].reshape(V, -1).double()
    for got, ref in ((out, ag.reshape(V, -1).double() @ T.t()), (da, gg.reshape(V, -1).double() @ T)):
        assert float((got - ref).norm() / ref.norm()) <= 1.3e-6
