"""Embedding and message widths: those whose tangent kernels are compiled for
the width (message width half of 32, 64 or 128) and others, against the oracle
in FP64: evaluation and the full parameter adjoint."""

import numpy as np
import pytest
import torch

import paper_1909_08423_amd as pn
from gpu_util import announce, parity_ratios
from oracle import Oracle
from synth.configs import NetShape, make_system_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dx,dz", [(32, 16), (64, 32), (128, 64), (32, 32), (64, 16), (128, 32), (64, 64)])
@pytest.mark.parametrize("n", [3, 7])
def test_widths(dx, dz, n):
    announce(f"widths {dx}/{dz}, H{n}")
    z = (np.arange(n) - (n - 1) / 2) * 1.8
    xyz = np.stack([np.zeros(n), np.zeros(n), z], 1)
    net = NetShape(16, 10.0, dx, dz, 2)
    w = make_system_workload(f"H{n}", xyz, [1] * n, (n + 1) // 2, n // 2, [4] * n, [0] * n, 4, net, 5, 1.0, dx + dz + n)
    ctx = pn.PauliNetContext(w.system, w.net)
    r = torch.tensor(w.walkers, dtype=torch.float64, device="cuda")
    th = torch.tensor(w.params, dtype=torch.float64, device="cuda")
    o = Oracle(w.system, w.net, w.params)
    out = {k: v.cpu().numpy() for k, v in ctx.eval(r, th, pn.PN_PREC_FP64).items()}
    ref = {k: v.numpy() for k, v in o.evaluate(w.walkers).items()}
    np.testing.assert_array_equal(out["sign"], ref["sign"])
    for k, v in parity_ratios(out, ref).items():
        assert v.max() <= 1e-6, f"{k}: worst {v.max():.3e}"
    if n == 3:
        ct = np.array([0.7, -1.3, 0.4, 1.1, -0.2])
        g = ctx.eval_backward(r, th, None, pn.PN_PREC_FP64, ct_lap=torch.tensor(ct, device="cuda")).cpu().numpy()
        gr = o.param_grad_full(w.walkers, ct_lap=ct).numpy()
        assert np.linalg.norm(g - gr) <= 1e-8 * np.linalg.norm(gr)


@pytest.mark.parametrize("n", [10, 12])
def test_full_adjoint_two_blocks_per_cu(n):
    """Chunks of the full adjoint that leave LDS for two 512-thread blocks."""
    announce(f"full adjoint, width 64, H{n}")
    z = (np.arange(n) - (n - 1) / 2) * 1.8
    xyz = np.stack([np.zeros(n), np.zeros(n), z], 1)
    net = NetShape(16, 10.0, 64, 32, 2)
    w = make_system_workload(f"H{n}", xyz, [1] * n, (n + 1) // 2, n // 2, [4] * n, [0] * n, 3, net, 2, 1.0, 5 * n)
    ctx = pn.PauliNetContext(w.system, w.net)
    r = torch.tensor(w.walkers, dtype=torch.float64, device="cuda")
    th = torch.tensor(w.params, dtype=torch.float64, device="cuda")
    ct = np.array([0.7, -1.3])
    g = ctx.eval_backward(r, th, None, pn.PN_PREC_FP64, ct_lap=torch.tensor(ct, device="cuda")).cpu().numpy()
    gr = Oracle(w.system, w.net, w.params).param_grad_full(w.walkers, ct_lap=ct).numpy()
    assert np.linalg.norm(g - gr) <= 1e-8 * np.linalg.norm(gr)
