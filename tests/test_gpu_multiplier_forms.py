"""GPU: the p x p algebra at the width from which it runs on the device, in the
forms that Algorithm PLAM (no normalization, Lambda0 as the multiplier) and the
SCF iteration (scales from the host) give it, against the oracle's iterations."""
import numpy as np
import pytest

import workloads as wl
from oracle import fem, pcal, scf

pytestmark = pytest.mark.gpu


def _problem(p, cells, scf_run):
    ax = wl.uniform_axis(-5.0, 5.0, cells)
    Z, R = np.array([6.0, 8.0]), np.array([[-1.1, 0.2, 0.1], [1.2, -0.3, 0.2]])
    w = wl.Workload("edge", wl.kuhn_mesh(ax, ax, ax), Z, R, p=p, beta=1.0, scf=scf_run, seed=0)
    return w, fem.discretize(w.mesh, Z, R)


def _compare(w, X0, hist, tol_kkt, tol_energy, **prm):
    import torch
    from paper_2007_14228_amd import Solver
    s = Solver()
    s.load_workload(w)
    s.set_params(beta=1.0, tol=1e-30, energy_every=1, max_iter=len(hist) - 1, **prm)
    s.set_x0(torch.from_numpy(X0).cuda(), orthonormalize=False)
    st, _, _ = s.step(len(hist))
    s.close()
    assert len(st) == len(hist)
    for a, b in zip(st, hist):
        assert abs(a["kkt"] - b.kkt) <= tol_kkt * b.kkt, (a, b)
        assert abs(a["fea"] - b.fea) <= tol_kkt * (b.fea + 1.0), (a, b)
        assert abs(a["energy"] - b.energy) <= tol_energy * abs(b.energy), (a, b)


@pytest.mark.parametrize("precond,step_rule,eta0", [("none", "fixed", 60.0), ("paper", "bb2", 0.0)])
@pytest.mark.parametrize("p", [63, 64, 65])
def test_plam(p, precond, step_rule, eta0):
    print(f"[gpu] multiplier plam p={p} {precond}", flush=True)
    w, d = _problem(p, 10, False)
    prob = pcal.LinearProblem(d.row_ptr, d.col, d.H, d.B, 0.5 * d.L)
    X0 = pcal.chol_gs(prob, wl.random_block(3, d.n, p))
    prm = dict(precond=precond, step_rule=step_rule, eta0=eta0, algorithm="plam")
    _, hist = pcal.pcal(prob, X0, pcal.Params(beta=1.0, tol=1e-30, max_iter=4, **prm))
    # as in PCAL: products of 1e-12 and a BB quotient of differences, five steps
    _compare(w, X0, hist, 1e-9, 1e-9, **prm)


@pytest.mark.parametrize("p", [63, 64, 65])
def test_scf(p):
    print(f"[gpu] multiplier scf p={p}", flush=True)
    w, d = _problem(p, 9, True)
    prob = scf.KSProblem(d, w.Z, w.R)
    X0 = pcal.chol_gs(pcal.LinearProblem(d.row_ptr, d.col, d.H, d.B, 0.5 * d.L), wl.random_block(3, d.n, p))
    _, hist = pcal.pcal(prob, X0, pcal.Params(beta=1.0, tol=1e-30, max_iter=3, precond="paper"))
    # the Hartree solves stop at 1e-12, each from its own start
    _compare(w, X0, hist, 1e-8, 1e-9, precond="paper", scf=1)
