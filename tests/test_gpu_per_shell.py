"""The per-shell SH kernels on tables that stay with them: two equal shells
whose slices are 16-byte pieces (96 directions), and unequal shells of more
directions than a row tile holds (524).  Large batches, so that FP32 Signal2SH
runs with resident tables and BF16 reductions over 65 .. 96 directions two
voxel blocks per wave; each against the FP64 oracle and against the kernels'
other forms (DLM_SHELL_RESIDENT=0, DLM_SHELL_PAIRS=0).
"""
import os

import numpy as np
import pytest
import torch

import datagen as dg
import paper_1808_01517_amd as dl
from oracle import sh as osh

from parity_util import check, fmt

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TABLES = {"equal": (96, 96), "unequal": (96, 128, 90, 110, 100)}


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


def plans(kind):
    dirs = [dg.perturb_directions(dg.fibonacci_hemisphere(n), 2.0, dg.rng_for(11, 0, s))
            for s, n in enumerate(TABLES[kind])]
    bvecs = np.concatenate([np.zeros((2, 3))] + dirs)
    bvals = np.concatenate([np.zeros(2)] + [np.full(d.shape[0], 1000.0 * (s + 1)) for s, d in enumerate(dirs)])
    return osh.SHPlan(bvecs, bvals, 8, 0.006), dl.SHPlan(bvecs, bvals, 8, 0.006)


def run(plan, x, c, prec):
    out = (dl.signal2sh_fwd(plan, x, precision=prec), dl.sh2signal_bwd(plan, x, precision=prec),
           dl.sh2signal_fwd(plan, c, precision=prec), dl.signal2sh_bwd(plan, c, precision=prec))
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("kind,V", [("equal", 140_003), ("equal", 1007), ("unequal", 270_021), ("unequal", 33)])
def test_against_oracle_and_other_forms(kind, V, prec):
    oplan, plan = plans(kind)
    rng = np.random.default_rng(97)
    c = rng.standard_normal((V, plan.n_shells, plan.K)).astype(np.float32).astype(np.float64)
    x = osh.sh2signal(oplan, rng.standard_normal(c.shape)).astype(np.float32).astype(np.float64)
    xg, cg = cuda(x), cuda(c)
    out = run(plan, xg, cg, prec)
    refs = (osh.signal2sh(oplan, x), osh.sh2signal_adjoint(oplan, x), osh.sh2signal(oplan, c),
            osh.signal2sh_adjoint(oplan, c))
    errs = {}
    for name, o, r in zip(("c", "dc", "x", "dx"), out, refs):
        check(name, o, r, prec, errs)
    print(f"[parity] per-shell kernels {kind} {prec}, V={V}: " + fmt(errs), flush=True)
    for switch in ("DLM_SHELL_RESIDENT", "DLM_SHELL_PAIRS"):
        os.environ[switch] = "0"
        try:
            other = run(plan, xg, cg, prec)
        finally:
            del os.environ[switch]
        for i, (a, b) in enumerate(zip(out, other)):
            if switch == "DLM_SHELL_RESIDENT" and i == 0:  # FP32's other form sums in another order
                check("c, other form", b, refs[0], prec)
            else:
                assert torch.equal(a, b), (switch, i)


# either side of the lines between whole rows and per-shell waves: call bytes
# from 8 to 128 MiB with 16-byte rows (two shells of 90, order 10, 1 248 bytes a
# voxel), from 32 MiB with long FP32 reductions (three of 90, order 8, 1 620
# bytes), below 128 MiB with short FP32 slices (three of 60, order 2, 792 bytes)
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("dirs,order,sizes", [((90, 90), 10, (6_721, 6_722, 107_546, 107_547)),
                                              ((90, 90, 90), 8, (20_712, 20_713, 82_850, 82_851)),
                                              ((60, 60, 60), 2, (65_535, 65_536, 169_466, 169_467))])
def test_lines_between_rows_and_shells(dirs, order, sizes, prec):
    tab = [dg.perturb_directions(dg.fibonacci_hemisphere(n), 2.0, dg.rng_for(12, 0, s)) for s, n in enumerate(dirs)]
    bvecs = np.concatenate(tab)
    bvals = np.concatenate([np.full(d.shape[0], 1000.0 * (s + 1)) for s, d in enumerate(tab)])
    oplan, plan = osh.SHPlan(bvecs, bvals, order, 0.006), dl.SHPlan(bvecs, bvals, order, 0.006)
    rng = np.random.default_rng(98)
    V = max(sizes)
    c = rng.standard_normal((V, plan.n_shells, plan.K)).astype(np.float32).astype(np.float64)
    x = osh.sh2signal(oplan, rng.standard_normal(c.shape)).astype(np.float32).astype(np.float64)
    xg, cg = cuda(x), cuda(c)
    refs = (osh.signal2sh(oplan, x), osh.sh2signal_adjoint(oplan, x), osh.sh2signal(oplan, c),
            osh.signal2sh_adjoint(oplan, c))
    for n in sizes:
        for name, o, r in zip(("c", "dc", "x", "dx"), run(plan, xg[:n], cg[:n], prec), refs):
            check(f"{name}, V={n}", o, r[:n], prec)
