"""GPU: what a step reports when the p x p quantities are not finite or a column
is zero, with the algebra on the host (p = 63) and on the device."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _solver(p, h_bad=None):
    import scipy.sparse as sp
    import torch
    from paper_2007_14228_amd import Solver
    n = 4 * p
    rng = np.random.default_rng(p)
    o = rng.uniform(-0.3, 0.3, n - 1)
    A = sp.diags([o, rng.uniform(1, 2, n), o], [-1, 0, 1]).tocsr()
    H = A.data.copy() if h_bad is None else np.full_like(A.data, h_bad)
    s = Solver()
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    s.csr_load(dev(A.indptr.astype(np.int64)), dev(A.indices.astype(np.int32)), dev(H), dev(A.data), dev(A.data))
    s.set_params(beta=1.0, tol=1e-30, max_iter=10, precond="none", step_rule="fixed", eta0=50.0)
    X = torch.from_numpy(rng.standard_normal((n, p))).cuda()
    return s, X


@pytest.mark.parametrize("p", [63, 64, 65, 300])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_the_matrix_that_is_not_finite_is_named(p, value):
    print(f"[gpu] multiplier errors p={p} {value}", flush=True)
    s, X = _solver(p, h_bad=value)
    s.set_x0(X)
    with pytest.raises(RuntimeError, match=r"non-finite X\^T H X") as e:
        s.step(1)
    assert e.value.code == -5
    s.close()


@pytest.mark.parametrize("p", [63, 64, 65])
def test_blocks_that_are_not_finite(p):
    """A start block taken as given is checked by its B-norms; an overflow on the way there is X^T B X's."""
    print(f"[gpu] multiplier block errors p={p}", flush=True)
    s, X = _solver(p)
    X = 1e200 * X          # finite, its squares are not
    with pytest.raises(RuntimeError) as e:
        s.set_x0(X, orthonormalize=False)
        s.step(1)
    assert e.value.code in (-5, -7) and ("X^T B X" in str(e.value) or "B-norm" in str(e.value)), str(e.value)
    s.close()
