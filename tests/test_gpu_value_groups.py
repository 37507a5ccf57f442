"""The value pass groups several walkers per block, the more the larger the
batch; a walker's outputs must not depend on the group it falls into, nor on
whether the derivative jets of the filters are computed beside the values."""

import numpy as np
import pytest
import torch

import paper_1909_08423_amd as pn
from synth import make_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("idx,n", [(1, 1025), (2, 771), (7, 1537), (5, 70)])
@pytest.mark.parametrize("prec", [pn.PN_PREC_FP64, pn.PN_PREC_NET_FP32])
def test_outputs_do_not_depend_on_the_group(idx, n, prec):
    w = make_config(idx, n_walkers=n)
    ctx = pn.PauliNetContext(w.system, w.net)
    r = torch.tensor(w.walkers, dtype=torch.float64, device="cuda")
    th = torch.tensor(w.params, dtype=torch.float64, device="cuda")
    whole = ctx.eval(r, th, prec)
    value = ctx.eval(r, th, prec, want_derivs=False)
    assert torch.equal(value["logabs"], whole["logabs"]) and torch.equal(value["sign"], whole["sign"])
    for lo, hi in ((0, 1), (n // 2, n // 2 + 5), (n - 3, n)):
        part = ctx.eval(r[lo:hi], th, prec)
        for k in part:
            assert torch.equal(part[k], whole[k][lo:hi]), (k, lo, hi)
    assert np.isfinite(whole["eloc"].cpu().numpy()).all()
