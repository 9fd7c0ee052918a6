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


def sums(x, T):
    """x @ T^T in float64, every product formed (0 * inf is NaN)."""
    with np.errstate(invalid="ignore"):
        return np.stack([(v.astype(np.float64) * T).sum(1) for v in x])


def same(out, ref):
    """float32's specials, and the finite entries to FP32's norm-wise bound."""
    out = out.double().cpu().numpy().reshape(ref.shape)
    assert np.array_equal(np.isnan(out), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(out[inf], ref[inf])
    fin = np.isfinite(ref)
    if fin.any():
        assert np.linalg.norm(out[fin] - ref[fin]) <= 1e-5 * np.linalg.norm(ref[fin])


@pytest.mark.parametrize("weights", ["finite", "nan"])
@pytest.mark.parametrize("layer", [(3, 32, 8, 300), (9, 3, 4, 70), (32, 3, 8, 1100), (13, 16, 2, 515)])
def test_rows_of_nan_among_others(layer, weights):
    # half of the voxels NaN, whole or in one value, infinities in a few others
    # and beside NaN, and (weights) an output channel of NaN weights: entries
    # that are NaN by their operands keep the first result, the rest of the same
    # tiles is float32's
    C, O, L, V = layer
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(90), L, L, (8, 8), np.deg2rad(30), 0.006)
    W = dg.lsc_weights(22, 0, C, O, plan.T)[0].astype(np.float32)
    if weights == "nan":
        W[O // 2] = np.nan
    _, Bnb, Pm = plan.tables()
    Q = np.einsum("ki,itj->tkj", Pm, Bnb.reshape(plan.m, plan.T, plan.K_in))
    T = np.einsum("oct,tkj->okcj", W.astype(np.float64), Q).reshape(O * plan.K_out, C * plan.K_in)
    rng = np.random.default_rng(22)
    x = {}
    for name, n in (("a", C * plan.K_in), ("g", O * plan.K_out)):
        v = rng.standard_normal((V, n)).astype(np.float32)
        v[1::4] = np.nan
        v[3::4, n - 1] = np.nan
        v[V // 2 // 4 * 4, n // 3] = np.inf
        v[8, 0], v[8, n - 1], v[11, 0], v[V - 1, n // 2] = np.inf, -np.inf, np.inf, -np.inf
        x[name] = v
    a, g = x["a"], x["g"]
    ag, gg, Wg = cuda(a.reshape(V, C, -1)), cuda(g.reshape(V, O, -1)), cuda(W)
    same(dl.lsc_fwd(plan, ag, Wg, None), sums(a, T))
    same(dl.lsc_bwd(plan, ag, Wg, gg, need_weight_grad=False, need_bias_grad=False)[0], sums(g, T.T))
    ai, gi = cuda(a.T[None]), cuda(g.T[None])
    same(dl.lsc_fwd_image(plan, ai, Wg)[0][0].t().contiguous(), sums(a, T))
    # masked by ReLU bits that the NaN, infinite and negative outputs leave clear
    out, bits = dl.lsc_fwd_image(plan, ai, Wg, relu=True, need_bits=True)
    with np.errstate(invalid="ignore"):
        gm = np.where(out[0].t().cpu().numpy() > 0, g, np.float32(0.0))
    da = dl.lsc_bwd_image(plan, ai, Wg, gi, bits, need_weight_grad=False, need_bias_grad=False)[0]
    same(da[0].t().contiguous(), sums(gm, T.T))


@pytest.mark.parametrize("case", [(130, 20, 700), (20, 145, 1500), (3, 2, 40)])
def test_weight_gradient_specials(case):
    # order 0: dW[o][c][t] = Q[t] sum_v g[v][o] a[v][c]
    C, O, V = case
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(12), 0, 0, (6,), np.deg2rad(30), 0.006)
    _, Bnb, Pm = plan.tables()
    q = np.einsum("ki,itj->t", Pm, Bnb.reshape(plan.m, plan.T, 1))
    rng = np.random.default_rng(23)
    a, g = (rng.standard_normal((V, n)).astype(np.float32) for n in (C, O))
    a[5, 1], a[30, C - 1], a[V - 1, 0], a[V - 2, 0] = np.nan, np.inf, np.inf, np.inf
    g[30, 0], g[12, O - 1], g[V - 3, O // 2] = 0.0, np.nan, -np.inf
    with np.errstate(invalid="ignore"):
        G = np.stack([(g[:, o, None].astype(np.float64) * a.astype(np.float64)).sum(0) for o in range(O)])
        ref = G[:, :, None] * q
        db = g.astype(np.float64).sum(0) * Pm.sum()
    W = cuda(dg.lsc_weights(23, 0, C, O, plan.T)[0])
    _, dW, b = dl.lsc_bwd(plan, cuda(a[:, :, None]), W, cuda(g[:, :, None]), need_input_grad=False)
    same(dW, ref)
    same(b, db)
    _, dW, b = dl.lsc_bwd_image(plan, cuda(a.T[None]), W, cuda(g.T[None]), need_input_grad=False)
    same(dW, ref)
    same(b, db)


@pytest.mark.parametrize("scale", [-90, -112, -120, -124])
@pytest.mark.parametrize("layer", [(3, 32, 8, 130), (9, 3, 4, 70), (32, 3, 8, 300)])
def test_values_below_the_parts(layer, scale):
    # operands whose third part lies under bfloat16's smallest number: the
    # bound is float32's, sqrt(K) / 2 roundings of 2^-24 of products that add up
    # at random (K up to 1440: 1.1e-6), and below 2^-121 the operand's spacing,
    # 2^-149, against its scale
    C, O, L, V = layer
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(90), L, L, (8, 8), np.deg2rad(30), 0.006)
    W = dg.lsc_weights(24, 0, C, O, plan.T)[0].astype(np.float32)
    _, Bnb, Pm = plan.tables()
    Q = np.einsum("ki,itj->tkj", Pm, Bnb.reshape(plan.m, plan.T, plan.K_in))
    rng = np.random.default_rng(24)
    s = 2.0 ** scale
    a, g = (rng.standard_normal((V, n)).astype(np.float32) for n in (C * plan.K_in, O * plan.K_out))
    at, gt = ((x.astype(np.float64) * s).astype(np.float32) for x in (a, g))
    a[::3], at[::3] = 0.0, 0.0  # zeros stay zeros
    tol = 1.1e-6 + 2.0 ** (-149 - scale)

    def close(out, ref):
        out = out.double().cpu().numpy().reshape(ref.shape) / s
        ref = ref / s
        assert np.linalg.norm(out - ref) <= tol * np.linalg.norm(ref)

    def grads(x, y):
        G = (y.astype(np.float64).T @ x.astype(np.float64)).reshape(O, plan.K_out, C, plan.K_in)
        return np.einsum("okcj,tkj->oct", G, Q)

    T = np.einsum("oct,tkj->okcj", W.astype(np.float64), Q).reshape(O * plan.K_out, C * plan.K_in)
    ac, gc, Wc = cuda(a.reshape(V, C, -1)), cuda(g.reshape(V, O, -1)), cuda(W)
    atc, gtc = cuda(at.reshape(V, C, -1)), cuda(gt.reshape(V, O, -1))
    close(dl.lsc_fwd(plan, atc, Wc, None), at.astype(np.float64) @ T.T)
    da, dW, _ = dl.lsc_bwd(plan, ac, Wc, gtc)
    close(da, gt.astype(np.float64) @ T)
    close(dW, grads(a, gt))
    close(dl.lsc_bwd(plan, atc, Wc, gc)[1], grads(at, g))
    out = dl.lsc_fwd_image(plan, cuda(at.T[None]), Wc)[0]
    close(out[0].t().contiguous(), at.astype(np.float64) @ T.T)
    da, dW, _ = dl.lsc_bwd_image(plan, cuda(a.T[None]), Wc, cuda(gt.T[None]))
    close(da[0].t().contiguous(), gt.astype(np.float64) @ T)
    close(dW, grads(a, gt))


@pytest.mark.parametrize("scale", [-90, -108, -118])
@pytest.mark.parametrize("layer", [(3, 32, 8, 130), (9, 3, 4, 70), (32, 3, 8, 300)])
def test_weights_below_the_parts(layer, scale):
    # the same of the weights: float32's roundings as above, and those of the
    # folded entries, sums of T products that each round to the float32 grid,
    # 2^-149 at the finest, against their root mean square
    C, O, L, V = layer
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(90), L, L, (8, 8), np.deg2rad(30), 0.006)
    s = 2.0 ** scale
    W = (dg.lsc_weights(25, 0, C, O, plan.T)[0].astype(np.float64) * s).astype(np.float32)
    _, Bnb, Pm = plan.tables()
    Q = np.einsum("ki,itj->tkj", Pm, Bnb.reshape(plan.m, plan.T, plan.K_in))
    T = np.einsum("oct,tkj->okcj", W.astype(np.float64) / s, Q).reshape(O * plan.K_out, C * plan.K_in)
    tol = 1.1e-6 + np.sqrt(plan.T) * 2.0 ** (-149 - scale) / np.sqrt(np.mean(T ** 2))
    rng = np.random.default_rng(25)
    a, g = (rng.standard_normal((V, n)).astype(np.float32) for n in (C * plan.K_in, O * plan.K_out))
    a[::3] = 0.0
    ac, gc, Wc = cuda(a.reshape(V, C, -1)), cuda(g.reshape(V, O, -1)), cuda(W)
    da = dl.lsc_bwd(plan, ac, Wc, gc, need_weight_grad=False, need_bias_grad=False)[0]
    im = dl.lsc_fwd_image(plan, cuda(a.T[None]), Wc)[0][0].t().contiguous()
    for out, ref in ((dl.lsc_fwd(plan, ac, Wc, None), a.astype(np.float64) @ T.T), (da, g.astype(np.float64) @ T),
                     (im, a.astype(np.float64) @ T.T)):
        out = out.double().cpu().numpy().reshape(ref.shape) / s
        assert np.linalg.norm(out - ref) <= tol * np.linalg.norm(ref)


@pytest.mark.parametrize("layer", [(3, 32, 16384), (32, 64, 2048)])
def test_a_background_of_nan_costs_little(layer):
    # 1.0 to 1.5 times the finite time; 25 to 40 times when every tile with such
    # a value is computed again
    C, O, V = layer
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(90), 8, 8, (8, 8), np.deg2rad(30), 0.006)
    W = cuda(dg.lsc_weights(26, 0, C, O, plan.T)[0])
    gen = torch.Generator(device=DEV).manual_seed(26)
    a, g = (torch.randn(V, n, plan.K_in, device=DEV, generator=gen) for n in (C, O))
    nan_a, nan_g = a.clone(), g.clone()
    nan_a[1::2], nan_g[1::2] = np.nan, np.nan

    def time(x, y):
        best = []
        for _ in range(7):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(4):
                dl.lsc_fwd(plan, x, W, None)
                dl.lsc_bwd(plan, x, W, y)
            t1.record()
            torch.cuda.synchronize()
            best.append(t0.elapsed_time(t1))
        return sorted(best)[3]

    assert time(nan_a, nan_g) <= 5 * time(a, g)
