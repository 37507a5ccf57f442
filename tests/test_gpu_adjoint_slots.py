"""Full adjoint where the members list the same orbitals in other slots, so
that successive members add to one table entry from different lanes: FP64
against the oracle's third-order autograd."""

import numpy as np
import pytest
import torch

import paper_1909_08423_amd as pn
from oracle import Oracle
from synth.configs import NetShape, make_system_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_up,n_down", [(5, 4), (9, 1), (16, 2)])
def test_full_adjoint_of_reordered_members(n_up, n_down):
    n = n_up + n_down
    w = make_system_workload(f"Z{n}", [[0.0, 0.0, 0.0]], [n], n_up, n_down, [8], [5], 7, NetShape(16, 10.0, 32, 16, 1), 2,
                             1.5, 300 + n)
    for dets in (w.system.det_up, w.system.det_down):
        for p in range(1, len(dets)):
            dets[p] = np.roll(dets[p], p)
    print(n_up, n_down, flush=True)
    ctx = pn.PauliNetContext(w.system, w.net)
    rng = np.random.default_rng(n)
    cg, cl = rng.standard_normal(w.walkers.shape), rng.standard_normal(2)
    dev = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda")  # noqa: E731
    g = ctx.eval_backward(dev(w.walkers), dev(w.params), None, pn.PN_PREC_FP64, ct_grad=dev(cg), ct_lap=dev(cl))
    ref = Oracle(w.system, w.net, w.params).param_grad_full(w.walkers, ct_grad=cg, ct_lap=cl).numpy()
    assert np.linalg.norm(g.cpu().numpy() - ref) <= 1e-8 * np.linalg.norm(ref)
