"""Systems whose value pass takes the message channels one after the other
through one LDS table (three do not fit a block of one walker): value-path
adjoint and nucleus-value gradient in FP64 against the oracle's autograd."""

import numpy as np
import pytest
import torch

import paper_1909_08423_amd as pn
from oracle import Oracle
from synth.configs import NetShape, make_system_workload

pytestmark = pytest.mark.gpu


def chain(n, net, walkers):
    z = (np.arange(n) - (n - 1) / 2) * 1.8
    xyz = np.stack([np.zeros(n), np.zeros(n), z], 1)
    return make_system_workload(f"H{n}", xyz, [1] * n, (n + 1) // 2, n // 2, [4] * n, [0] * n, 4, net, walkers, 1.0,
                                177 + n)


def dev(x):
    return torch.tensor(x, dtype=torch.float64, device="cuda")


# the first size past three tables, the last that took one wide table, the largest
@pytest.mark.parametrize("n,net", [
    (43, NetShape(16, 10.0, 128, 64, 2)),
    (48, NetShape(16, 10.0, 128, 64, 1)),
    (64, NetShape(16, 10.0, 64, 64, 2)),
])
def test_value_adjoint_one_message_table(n, net):
    print("value adjoint", n, net, flush=True)
    w = chain(n, net, 2)
    ctx = pn.PauliNetContext(w.system, w.net)
    ct = np.array([1.0, -0.7])
    g = ctx.eval_backward(dev(w.walkers), dev(w.params), dev(ct), pn.PN_PREC_FP64).cpu().numpy()
    ref = Oracle(w.system, w.net, w.params).param_grad_logabs(w.walkers, ct).numpy()
    assert np.linalg.norm(g - ref) <= 1e-8 * np.linalg.norm(ref)
    for name, off, shape in ctx.param_layout():
        k = slice(off, off + int(np.prod(shape)))
        assert np.linalg.norm(g[k] - ref[k]) <= 1e-8 * np.linalg.norm(ref), name


@pytest.mark.parametrize("n,net", [(31, NetShape(16, 10.0, 128, 128, 2)), (48, NetShape(16, 10.0, 128, 128, 1)),
                                   (47, NetShape(16, 10.0, 32, 128, 2))])
def test_nucleus_value_gradient_one_message_table(n, net):
    print("nucleus values", n, net, flush=True)
    w = make_system_workload(f"Z{n}", [[0.0, 0.0, 0.0]], [n], (n + 1) // 2, n // 2, [20], [8], 4, net, 2, 1.5, 277 + n)
    r = w.walkers.copy()
    r[0, 0] = 0.05 * np.array([0.6, -0.48, 0.64])
    r[1, 3] = 0.03 * np.array([0.64, -0.48, 0.6])
    ct = np.array([1.0, -0.7])
    ctx = pn.PauliNetContext(w.system, w.net)
    g = ctx.eval_backward_cusp(dev(r), dev(w.params), dev(ct), pn.PN_PREC_FP64).cpu().numpy()
    ref = Oracle(w.system, w.net, w.params).cusp_value_grad(r, ct).numpy()
    assert np.abs(ref).max() > 0
    assert np.linalg.norm(g - ref) <= 1e-8 * np.linalg.norm(ref)
