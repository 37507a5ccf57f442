"""Spin blocks around the 16 x 16 tiles of the determinant kernels (9 to 16
electrons of a spin, equal and unequal, and beyond), member by member: values,
derivatives and the full parameter adjoint against the oracle in FP64."""

import numpy as np
import pytest
import torch

import paper_1909_08423_amd as pn
from oracle import Oracle
from synth.configs import NetShape, make_system_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [17, 31, 34])
def test_member_by_member_determinants(n):
    z = (np.arange(n) - (n - 1) / 2) * 1.8
    xyz = np.stack([np.zeros(n), np.zeros(n), z], 1)
    net = NetShape(16, 10.0, 32, 16, 1, 4)  # PN_DET_DIRECT
    w = make_system_workload(f"H{n}", xyz, [1] * n, (n + 1) // 2, n // 2, [4] * n, [0] * n, 3, net, 2, 1.0, 7 + n)
    ctx = pn.PauliNetContext(w.system, w.net)
    r = torch.tensor(w.walkers, dtype=torch.float64, device="cuda")
    th = torch.tensor(w.params, dtype=torch.float64, device="cuda")
    out = {k: v.cpu().numpy() for k, v in ctx.eval(r, th, pn.PN_PREC_FP64).items()}
    o = Oracle(w.system, w.net, w.params)
    ref = {k: v.numpy() for k, v in o.evaluate(w.walkers).items()}
    assert np.array_equal(out["sign"], ref["sign"])
    assert np.all(np.abs(out["logabs"] - ref["logabs"]) <= 1e-6 * np.maximum(1, np.abs(ref["logabs"])))
    assert np.linalg.norm(out["grad"] - ref["grad"]) <= 1e-6 * np.linalg.norm(ref["grad"])
    scale = np.abs(ref["lap"]) + (ref["grad"] ** 2).sum((1, 2))
    assert np.all(np.abs(out["lap"] - ref["lap"]) <= 1e-6 * scale)
    assert np.all(np.abs(out["eloc"] - ref["eloc"]) <= 1e-6 * scale)
    ct = np.array([0.7, -1.3])
    g = ctx.eval_backward(r, th, torch.tensor(ct, device="cuda"), pn.PN_PREC_FP64).cpu().numpy()
    gr = o.param_grad_logabs(w.walkers, ct).numpy()
    assert np.linalg.norm(g - gr) <= 1e-8 * np.linalg.norm(gr)
    if n <= 18:
        g = ctx.eval_backward(r, th, None, pn.PN_PREC_FP64, ct_lap=torch.tensor(ct, device="cuda")).cpu().numpy()
        gr = o.param_grad_full(w.walkers, ct_lap=ct).numpy()
        assert np.linalg.norm(g - gr) <= 1e-8 * np.linalg.norm(gr)
