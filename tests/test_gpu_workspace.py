"""Folded LSC calls in a caller's workspace that starts at any dword: the
forward, the input gradient with and without each mask, and the weight
gradient, held to the FP64 oracle.  Tables that the streaming core does not
take at that address go to the register-staged core in float32.
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


def workspace_at(plan, C, O, prec, offset):
    """A workspace of exactly the bytes asked for, `offset` beyond an aligned address."""
    n = dl.lsc_workspace_bytes(plan, C, O, 1, prec, "folded")
    ws = dl.Workspace(n + 16, DEV)
    ws.buf = ws.buf[offset:offset + n]
    assert ws.buf.data_ptr() % 16 == offset
    return ws


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("offset", [0, 4, 8, 12])
@pytest.mark.parametrize("layer", [(3, 32, 8, 70), (32, 3, 8, 33), (1, 2, 0, 5), (2, 5, 2, 129)])
def test_folded_calls_at_any_dword(layer, offset, prec):
    C, O, L, V = layer
    g = dg.fibonacci_hemisphere(90)
    plan = dl.LSCPlan(g, L, L, (8, 8), np.deg2rad(30), 0.006)
    oplan = olsc.LSCPlan(g, L, L, (8, 8), np.deg2rad(30), 0.006)
    W, b = (x.astype(np.float32).astype(np.float64) for x in dg.lsc_weights(12, 0, C, O, plan.T))
    rng = np.random.default_rng(12)
    a = rng.standard_normal((V, C, plan.K_in)).astype(np.float32).astype(np.float64)
    da_out = rng.standard_normal((V, O, plan.K_out)).astype(np.float32).astype(np.float64)
    ws = workspace_at(plan, C, O, prec, offset)
    for relu in (False, True):
        ref, z = olsc.lsc_forward(oplan, a, W, b, relu)
        out = dl.lsc_fwd(plan, cuda(a), cuda(W), cuda(b), relu=relu, precision=prec, workspace=ws)
        check("out", out, ref, prec)
        mask = cuda(np.where(np.asarray(z) > 0, 1.0, 0.0).reshape(V, O, plan.K_out))  # the oracle's ReLU pattern
        da_ref, dW_ref, db_ref = olsc.lsc_backward(oplan, a, W, z, da_out, relu)
        for relu_in in (False, True):
            da, dW, db = dl.lsc_bwd(plan, cuda(a), cuda(W), cuda(da_out), a_out=mask, relu=relu, relu_in=relu_in,
                                    precision=prec, workspace=ws)
            check("da", da, da_ref * (a > 0) if relu_in else da_ref, prec)
            check("dW", dW, dW_ref, prec, kind="sum")
            check("db", db, db_ref, prec, kind="sum")


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_images_and_bits_refuse_before_any_launch(prec):
    C, O, P = 2, 16, 40
    plan = dl.LSCPlan(dg.fibonacci_hemisphere(30), 2, 2, (6,), np.deg2rad(30), 0.006)
    L, code = dl.lib(), dl.precision_code(prec)
    gen = torch.Generator(device=DEV).manual_seed(13)
    a, g = (torch.randn(1, n * plan.K_in, P, device=DEV, generator=gen) for n in (C, O))
    W = torch.randn(O, C, plan.T, device=DEV, generator=gen)
    out, da, dW = torch.zeros_like(g), torch.zeros_like(a), torch.zeros_like(W)
    bits = torch.zeros((P, O * plan.K_out // 16), dtype=torch.int16, device=DEV)
    ws = workspace_at(plan, C, O, prec, 4)
    ws.buf.zero_()
    st = torch.cuda.current_stream().cuda_stream
    calls = [
        L.dlm_lsc_fwd_image(plan.handle, a.data_ptr(), C, W.data_ptr(), None, O, out.data_ptr(), 1, P, 0, None, ws.ptr(),
                            ws.nbytes, code, st),
        L.dlm_lsc_bwd_image(plan.handle, a.data_ptr(), C, W.data_ptr(), O, None, g.data_ptr(), da.data_ptr(),
                            dW.data_ptr(), None, 1, P, ws.ptr(), ws.nbytes, code, st),
        L.dlm_lsc_fwd_io(plan.handle, a.data_ptr(), C, W.data_ptr(), None, O, out.data_ptr(), P, 1, 0, bits.data_ptr(),
                         dl.form_code("folded"), ws.ptr(), ws.nbytes, code, st),
    ]
    torch.cuda.synchronize()
    assert calls == [dl._lib.DLM_EINVAL] * 3
    for t in (out, da, dW, bits, ws.buf):
        assert not t.any()
