"""GPU: steps at the width from which the p x p algebra runs on the device, on
both sides of it and at broken and whole multiples of its block, in both
algorithms, against the oracle's iteration (FP64: 1e-9 relative after five
steps, as products of 1e-12 and a BB quotient of differences leave)."""
import numpy as np
import pytest

import workloads as wl
from oracle import fem, pcal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [63, 64, 65, 256, 257])
def test_steps_follow_the_oracle(p):
    import torch
    from paper_2007_14228_amd import Solver
    print(f"[gpu] multiplier edges p={p}", flush=True)
    ax = wl.uniform_axis(-5.0, 5.0, 10)
    Z, R = np.array([6.0, 8.0]), np.array([[-1.1, 0.2, 0.1], [1.2, -0.3, 0.2]])
    w = wl.Workload("edge", wl.kuhn_mesh(ax, ax, ax), Z, R, p=p, beta=1.0, scf=False, seed=0)
    d = fem.discretize(w.mesh, Z, R)
    prob = pcal.LinearProblem(d.row_ptr, d.col, d.H, d.B, 0.5 * d.L)
    X0 = pcal.chol_gs(prob, wl.random_block(3, d.n, p))
    _, hist = pcal.pcal(prob, X0, pcal.Params(beta=1.0, tol=1e-30, max_iter=4, precond="paper"))
    s = Solver()
    s.load_workload(w)
    s.set_params(beta=1.0, tol=1e-30, max_iter=4, precond="paper", energy_every=1)
    s.set_x0(torch.from_numpy(X0).cuda(), orthonormalize=False)
    st, _, _ = s.step(5)
    assert len(st) == len(hist) == 5
    for a, b in zip(st, hist):
        assert abs(a["kkt"] - b.kkt) <= 1e-9 * b.kkt, (a, b)
        assert abs(a["energy"] - b.energy) <= 1e-9 * abs(b.energy), (a, b)
    s.close()
