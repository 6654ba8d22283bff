"""GPU: a context takes its blocks over from one start block to the next of the
same shape.  Whatever it ran before, a run from a start block gives the same
bits as on a fresh context."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def _run(s, X0, prm, steps):
    import torch
    s.set_params(**prm)
    s.set_x0(torch.from_numpy(X0).to("cuda"), orthonormalize=True)
    sts, _, _ = s.step(steps)
    return [(t["energy"], t["kkt"], t["precision"]) for t in sts], s.get_x().cpu().numpy()


def test_runs_on_kept_blocks_match_fresh_ones():
    from paper_2007_14228_amd import Solver
    w = wl.make_workload("c1")
    f64 = dict(beta=w.beta, tol=1e-30, max_iter=100, pcg_iters=4, energy_every=1, precond="paper", precision="f64",
               refine_tol=0.0)
    f32 = dict(f64, precision="f32")
    mixed = dict(f64, precision="f32", refine_tol=0.9)       # goes over to FP64 within its steps

    def fresh():
        s = Solver()
        s.load_workload(w)
        return s

    X = {p: wl.random_block(p, w.mesh.n_dofs, p) for p in (3, 5)}
    runs = [(f64, 3), (f64, 3), (f32, 3), (f32, 3), (mixed, 3), (mixed, 3), (f32, 3), (f32, 5), (f64, 5), (f64, 5)]
    s = fresh()
    for k, (prm, p) in enumerate(runs):
        print(f"[gpu] kept blocks, run {k}", flush=True)
        other = fresh()
        got, want = _run(s, X[p], prm, 5), _run(other, X[p], prm, 5)
        assert got[0] == want[0]
        assert np.array_equal(got[1], want[1])
        other.close()
    s.close()
