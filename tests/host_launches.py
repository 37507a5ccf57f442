"""What the library would launch, without a device: fake_hip.c in place of the
HIP runtime.  Run as a program of its own (the stand-in has to be loaded
before the library, and no real runtime beside it):

    python host_launches.py FAKE_SO  < calls.json  > results.json

A call is [system, net, walkers, precision, kind]; system = [n_up, n_down,
n_nuc, n_mo, n_det], net = [K, D_x, D_z, layers, flags].  A result holds the
status, the number of launches, those beyond the hardware limits, and for kind
"bytes" the workspace of the adjoints, of a VMC step and of an evaluation.
"""

import ctypes
import importlib.util
import json
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Fields:
    def __init__(self, **kw):
        self.__dict__.update(kw)


def binding():
    path = os.path.join(ROOT, "paper_1909_08423_amd", "_lib.py")
    spec = importlib.util.spec_from_file_location("paulinet_binding", path)  # without the package: no torch
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def system(n_up, n_down, n_nuc, n_mo, n_det):
    """A chain with s shells; members beyond the first replace the last
    orbital of the up spin."""
    per = -(-n_mo // n_nuc)
    n_shell = n_nuc * per
    up = np.tile(np.arange(n_up, dtype=np.int32), (n_det, 1))
    if n_up and n_mo > n_up:
        up[1:, -1] = n_up + np.arange(n_det - 1) % (n_mo - n_up)
    return Fields(nuc_xyz=np.outer(np.arange(n_nuc), [0.0, 0.0, 1.8]), charge=np.ones(n_nuc), n_up=n_up, n_down=n_down,
                  shell_center=np.repeat(np.arange(n_nuc), per), shell_l=np.zeros(n_shell),
                  shell_exp=np.linspace(0.5, 3.0, n_shell),
                  mo_coeff=np.random.default_rng(n_mo).standard_normal((n_shell, n_mo)), det_up=up,
                  det_down=np.tile(np.arange(n_down, dtype=np.int32), (n_det, 1)), ci=np.ones(n_det), cusp_radius=0.1,
                  cusp_nuc_value=None)


def main():
    fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    m = binding()
    lib = m.load_library()
    p, none, big = ctypes.c_void_p(1 << 20), ctypes.c_void_p(0), ctypes.c_size_t(1 << 50)
    results, contexts = [], {}
    for sys_args, net_args, nw, prec, kind in json.load(sys.stdin):
        key = json.dumps([sys_args, net_args])
        if key not in contexts:
            net = dict(zip(("n_feat", "dim_x", "dim_z", "n_layers", "flags"), net_args), feat_cutoff=10.0)
            contexts[key] = m.PauliNetContext(system(*sys_args), Fields(**net))
        ctx = contexts[key]
        c = ctx._ctx
        if kind == "bytes":
            results.append([ctx.plan(nw, prec, m.PLAN_VALUE_ADJOINT)["workspace_bytes"],
                            ctx.plan(nw, prec, m.PLAN_FULL_ADJOINT)["workspace_bytes"],
                            m.vmc_workspace_bytes(ctx, min(nw, 16384), prec),
                            ctx.plan(nw, prec, m.PLAN_EVAL)["workspace_bytes"]])
            continue
        job = m.pn_vmc_job(nw, *[p] * 6, 1, 0)
        slot = m.pn_job_slot(c, job, p, big.value)
        hp = m.pn_vmc_hparams(*m.DEFAULT_HPARAMS.values())
        fake.fake_reset()
        st = {
            "value": lambda: lib.pn_eval(c, none, nw, p, p, prec, p, p, none, none, none, p, big),
            "eval": lambda: lib.pn_eval(c, none, nw, p, p, prec, p, p, p, p, p, p, big),
            "noalloc": lambda: lib.pn_eval_noalloc(c, none, nw, p, p, prec, p, p, p, p, p),
            "adjoint": lambda: lib.pn_eval_backward(c, none, nw, p, p, prec, p, none, none, none, p, p, big),
            "full": lambda: lib.pn_eval_backward(c, none, nw, p, p, prec, p, p, p, none, p, p, big),
            "vmc": lambda: lib.pn_vmc_step(c, none, ctypes.byref(job), prec, ctypes.byref(hp), p, big),
            "serve": lambda: lib.pn_serve_step(none, ctypes.byref(slot), 1, prec, ctypes.byref(hp)),
            "langevin": lambda: lib.pn_langevin_run(c, none, nw, p, p, prec,
                                                    ctypes.byref(m.pn_langevin_hparams(0.57, 1.0)), p, 2, 1, 0, p, p, big),
            "cusp": lambda: lib.pn_eval_backward_cusp(c, none, nw, p, p, prec, p, p, p, big),
        }[kind]()
        beyond = []
        name, dims, lds, refused = ctypes.c_char_p(), (ctypes.c_uint32 * 6)(), ctypes.c_uint64(), ctypes.c_int()
        for k in range(fake.fake_count()):
            fake.fake_get(k, ctypes.byref(name), dims, ctypes.byref(lds), ctypes.byref(refused))
            if refused.value:
                beyond.append([name.value.decode(), list(dims), lds.value])
        results.append([st, fake.fake_count(), beyond])
    json.dump(results, sys.stdout)


if __name__ == "__main__":
    main()
