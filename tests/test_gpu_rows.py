"""SH transforms on whole voxel rows (csrc/rows.hip) where a tile or a run
ends: batches around 32 voxels, tensors that start at any float, shells of
unequal and odd sizes, tables at and beyond what one launch takes, raw
acquisitions with b = 0 volumes among the others.  The reference is the plan's
own float64 tables.
"""
import numpy as np
import pytest
import torch

import datagen as dg
import paper_1808_01517_amd as dl

from parity_util import check

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _plan(dirs, L, n_b0=0, seed=0):
    rng = np.random.default_rng(seed)
    g = np.concatenate([dg.fibonacci_hemisphere(n) + rng.uniform(-0.01, 0.01, (n, 3)) for n in dirs])
    b = np.concatenate([np.full(n, 1000.0 * (k + 1)) for k, n in enumerate(dirs)])
    if n_b0:  # b = 0 volumes spread through the acquisition, shells interleaved
        order = rng.permutation(len(b) + n_b0)
        g = np.concatenate([np.zeros((n_b0, 3)), g])[order]
        b = np.concatenate([np.zeros(n_b0), b])[order]
    return dl.SHPlan(g, b, L, 0.006), g, b


def at(offset, a):
    """a on the device, `offset` floats beyond the start of an allocation."""
    buf = torch.empty(offset + a.size, dtype=torch.float32, device=DEV)
    t = buf[offset:].view(a.shape)
    t.copy_(torch.from_numpy(a))
    return t


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("table", [
    ((6,), 2), ((30,), 4), ((45, 17, 31), 2), ((90, 90, 90), 8), ((96, 90), 12), ((128,), 8),
    ((30,) * 8, 4),            # 8 shells x 2 (30 directions) = 16 units, x 1 (15 coefficients)
    ((90,) * 4, 8),            # 24 units of directions: the most one launch takes
    ((90,) * 5, 8),            # 30: the tiled core
    ((130,), 8), ((16,) * 17, 4),
])
def test_transforms(table, prec):
    dirs, L = table
    plan, _, _ = _plan(dirs, L)
    mats = [plan.matrices(s) for s in range(plan.n_shells)]
    rng = np.random.default_rng(1)
    for V, off in ((1, 0), (31, 1), (32, 2), (33, 3), (100, 0)):
        x = (rng.random((V, plan.n_dw)) + 0.1).astype(np.float32)
        c = rng.standard_normal((V, plan.n_shells, plan.K)).astype(np.float32)
        xs = np.split(x.astype(np.float64), np.cumsum(dirs)[:-1], axis=1)
        c64 = c.astype(np.float64)
        fit = np.stack([xs[s] @ P.T for s, (_, P) in enumerate(mats)], 1)
        ev = np.concatenate([c64[:, s] @ B.T for s, (B, _) in enumerate(mats)], 1)
        fit_t = np.concatenate([c64[:, s] @ P for s, (_, P) in enumerate(mats)], 1)
        ev_t = np.stack([xs[s] @ B for s, (B, _) in enumerate(mats)], 1)
        check("signal2sh", dl.signal2sh_fwd(plan, at(off, x), precision=prec), fit, prec)
        check("sh2signal", dl.sh2signal_fwd(plan, at(off, c), precision=prec), ev, prec)
        check("signal2sh adjoint", dl.signal2sh_bwd(plan, at(off, c), precision=prec), fit_t, prec)
        check("sh2signal adjoint", dl.sh2signal_bwd(plan, at(off, x), precision=prec), ev_t, prec)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("table", [((30,), 4, 1), ((45, 17, 31), 2, 5), ((90, 90, 90), 8, 18), ((90,) * 5, 8, 60),
                                   ((128, 120, 110, 100), 8, 50)])
def test_raw(table, prec):
    dirs, L, n_b0 = table
    plan, _, b = _plan(dirs, L, n_b0)
    rng = np.random.default_rng(2)
    for V, off in ((1, 3), (33, 0), (70, 1)):
        raw = (rng.random((V, plan.n_total)) + 0.5).astype(np.float32) * 300
        norm = raw.astype(np.float64) / raw[:, b < 50].astype(np.float64).mean(1, keepdims=True)
        ref = np.stack([norm[:, plan.shells[s][2]] @ plan.matrices(s)[1].T for s in range(plan.n_shells)], 1)
        check("raw", dl.signal2sh_fwd_raw(plan, at(off, raw), precision=prec), ref, prec)


def test_specials_stay_in_their_voxel():
    plan, _, _ = _plan((30, 45), 4)
    x = torch.rand(70, plan.n_dw, device=DEV) + 0.1
    clean = dl.signal2sh_fwd(plan, x)
    x[5, 3], x[40, 29], x[69, 74] = float("nan"), float("inf"), float("nan")
    out = dl.signal2sh_fwd(plan, x)
    assert torch.isnan(out[5, 0]).all() and not torch.isfinite(out[40, 0]).any() and torch.isnan(out[69, 1]).all()
    out[5, 0], out[40, 0], out[69, 1] = clean[5, 0], clean[40, 0], clean[69, 1]
    assert torch.equal(out, clean)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("table", [
    ((30, 2), 0),              # two entries a voxel on one side
    ((30, 18), 2),             # 48 volumes padded in LDS, 12 coefficients not
    ((96, 64), 6),             # 160 and 56: padded on both sides
    ((96, 96, 96), 8),         # equal shells of whole 16-byte pieces: both kernels
    ((91,), 6), ((60,), 6),    # one shell, one side or both in 16-byte pieces
    ((30, 31, 32), 2),
])
def test_strides_and_groups(table, prec):
    # batches on either side of the second, third and fourth group of 32 voxels
    # a block and of the voxel count that decides for equal shells
    dirs, L = table
    plan, _, _ = _plan(dirs, L)
    mats = [tuple(torch.from_numpy(np.array(m)).double().to(DEV) for m in plan.matrices(s)) for s in range(plan.n_shells)]
    gen = torch.Generator(device=DEV).manual_seed(7)
    for V, off in ((65535, 0), (65536 + 33, 0), (98304 + 95, 1), (131072 + 1, 0)):
        x = torch.rand(off + V * plan.n_dw, device=DEV, generator=gen)[off:].view(V, plan.n_dw)
        c = torch.randn(off + V * plan.n_shells * plan.K, device=DEV, generator=gen)[off:].view(V, plan.n_shells, plan.K)
        xs = torch.split(x.double(), list(dirs), dim=1)
        fit = torch.stack([xs[s] @ P.t() for s, (_, P) in enumerate(mats)], 1)
        ev = torch.cat([c[:, s].double() @ B.t() for s, (B, _) in enumerate(mats)], 1)
        check("signal2sh", dl.signal2sh_fwd(plan, x, precision=prec), fit, prec)
        check("sh2signal", dl.sh2signal_fwd(plan, c, precision=prec), ev, prec)
