"""GPU: the inner CG of FP32 blocks at the edges of its form (one, two, three and
ten steps; single, two and four values an access; columns that are left as they
are; both product kernels) and where a step solves most of the system (beta
from the real sums): two iterations in FP32 against the same in FP64."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def _after_two(s, X, p, m, mode, precision):
    s.set_params(beta=1.0, tol=1e-30, max_iter=2, precond="paper", pcg_iters=m, precision=precision, spmm_mode=mode)
    s.set_x0(X)
    st, _, _ = s.step(3)
    return [x["kkt"] for x in st], s.get_x().cpu().numpy()


def _check(s, X, p, m, mode):
    k64, X64 = _after_two(s, X, p, m, mode, "f64")
    k32, X32 = _after_two(s, X, p, m, mode, "f32")
    # FP32 gradients lose two digits to the cancellation in H X - B X Lambda
    assert np.allclose(k32, k64, rtol=2e-5, atol=0), (m, k32, k64)
    assert np.linalg.norm(X32 - X64) <= 2e-5 * np.linalg.norm(X64), (m, np.linalg.norm(X32 - X64))


@pytest.mark.parametrize("mode", ["gather", "halo"])
@pytest.mark.parametrize("p", [1, 3, 6, 33, 64, 100])
def test_two_iterations(p, mode):
    import torch
    from paper_2007_14228_amd import Solver
    ax = wl.uniform_axis(-5.0, 5.0, 11)
    s = Solver()
    s.load_workload(wl.Workload("edge", wl.kuhn_mesh(ax, ax, ax), np.array([6.0, 8.0]),
                                np.array([[-1.1, 0.2, 0.1], [1.2, -0.3, 0.2]]), p=p, beta=1.0, scf=False, seed=0))
    X = torch.from_numpy(wl.random_block(3, s.n, p)).cuda()
    for m in (1, 2, 3, 10):
        print(f"[gpu] f32 cg p={p} m={m} {mode}", flush=True)
        _check(s, X, p, m, mode)
    s.close()


@pytest.mark.parametrize("mode", ["gather", "halo"])
@pytest.mark.parametrize("p", [3, 6, 64])
def test_steps_that_end_most_of_the_system(p, mode):
    """Small off-diagonals: a step lowers <r, z> to some 3e-4 of itself, so every
    beta comes from the real sums; without it the second step would be off by as
    much of P, which the first iteration takes whole."""
    import scipy.sparse as sp
    import torch
    from paper_2007_14228_amd import Solver
    n = 2000
    rng = np.random.default_rng(p)
    o = 0.08 * rng.uniform(-1, 1, n - 1)
    A = sp.diags([o, rng.uniform(1, 2, n), o], [-1, 0, 1]).tocsr()
    rows = np.repeat(np.arange(n), np.diff(A.indptr))
    B = np.where(A.indices == rows, 1.0, 0.0)
    H = A.data - 5.0 * B                       # bound states, so that every column takes the preconditioner
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    s = Solver()
    s.csr_load(dev(A.indptr.astype(np.int64)), dev(A.indices.astype(np.int32)), dev(H), dev(B), dev(A.data))
    X = dev(rng.standard_normal((n, p)))
    for m in (1, 2, 3, 40):
        print(f"[gpu] f32 cg nearly diagonal p={p} m={m} {mode}", flush=True)
        _check(s, X, p, m, mode)
    s.close()
