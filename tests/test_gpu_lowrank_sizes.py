"""The low-rank determinant path by spin size (each size up to eight electrons
of a spin has its own blocking) and by excitation rank (two orbitals of a spin,
or up to four), against the member-by-member path in FP64.

The bar is that of the other comparison of the two paths: per walker ratios
<= 1e-6, signs equal."""

import dataclasses

import numpy as np
import pytest
import torch

import paper_1909_08423_amd as pn
from gpu_util import announce, parity_ratios
from synth.configs import NetShape, make_system_workload, param_count

pytestmark = pytest.mark.gpu


def _workload(n, rank, n_det, walkers):
    z = (np.arange(n) - (n - 1) / 2) * 1.8
    xyz = np.stack([np.zeros(n), np.zeros(n), z], 1)
    net = NetShape(16, 10.0, 32, 16, 1)
    n_up, n_dn = (n + 1) // 2, n // 2
    w = make_system_workload(f"H{n}", xyz, [1] * n, n_up, n_dn, [4] * n, [0] * n, 3, net, walkers, 1.0, 11 * n + rank)
    rng = np.random.default_rng([n, rank])
    n_mo = n_up + 5

    def occupation(n_el, k):
        keep = set(range(n_el)) - set(rng.permutation(n_el)[:k].tolist())
        return sorted(keep | set((n_el + rng.permutation(n_mo - n_el)[:k]).tolist()))

    up, dn = [list(range(n_up))], [list(range(n_dn))]
    for p in range(1, n_det):
        up.append(occupation(n_up, min(rank if p == 1 else p % (rank + 1), n_up)))
        dn.append(occupation(n_dn, min((p // 2) % (rank + 1), n_dn)))
    mo = rng.standard_normal((w.system.mo_coeff.shape[0], n_mo))
    system = dataclasses.replace(w.system, det_up=np.array(up, w.system.det_up.dtype),
                                 det_down=np.array(dn, w.system.det_down.dtype),
                                 ci=np.concatenate([[1.0], rng.uniform(-0.3, 0.3, n_det - 1)]), mo_coeff=mo)
    params = 0.1 * rng.standard_normal(param_count(system.n_nuc, n_mo, net))
    return system, net, params, w.walkers


@pytest.mark.parametrize("n,n_det", [(4, 3), (9, 16), (11, 33), (14, 64), (15, 63), (16, 5), (19, 20)])
@pytest.mark.parametrize("rank", [2, 4])
def test_lowrank_against_members(n, n_det, rank):
    announce(f"low-rank against member by member: H{n}, {n_det} members of rank {rank}")
    system, net, params, walkers = _workload(n, rank, n_det, 67)
    out = []
    for flags in (0, pn._lib.PN_DET_DIRECT):
        ctx = pn.PauliNetContext(system, dataclasses.replace(net, flags=flags))
        assert bool(ctx.plan(67, pn.PN_PREC_FP64)["lowrank"]) == (flags == 0)
        r = torch.tensor(walkers, dtype=torch.float64, device="cuda")
        th = torch.tensor(params, dtype=torch.float64, device="cuda")
        out.append({k: v.cpu().numpy() for k, v in ctx.eval(r, th, pn.PN_PREC_FP64).items()})
    a, b = out
    np.testing.assert_array_equal(a["sign"], b["sign"])
    for k, v in parity_ratios(a, b).items():
        assert v.max() <= 1e-6, f"{k}: worst {v.max():.3e}"
