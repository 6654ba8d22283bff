"""GPU: the learned preconditioners' kernels at the edges of their column
mappings (a column a block, fewer columns than lanes, whole and broken row
groups, more columns than a block has threads) against the oracles.  The
networks run in FP32: an error of a few 1e-7 in a unit's tanh, 32 units with
weights below 1, relative to the largest value of the block: 2e-5 as in the
other tests of these networks."""
import numpy as np
import pytest

import workloads as wl
from oracle import fem, gnn, mlp

pytestmark = pytest.mark.gpu
NORM = np.array([-1.0, -2.0, -1.0, 0.0, 1.0, 1.5, 2.0, 1.0])


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.fixture(scope="module")
def system():
    from paper_2007_14228_amd import Solver
    ax = wl.uniform_axis(-4.0, 4.0, 10)
    w = wl.Workload("edge", wl.kuhn_mesh(ax, ax, ax), np.array([3.0]), np.array([[0.31, 0.17, 0.23]]), p=1, beta=1.0,
                    scf=False, seed=0)
    d = fem.discretize(w.mesh, w.Z, w.R)
    s = Solver()
    s.load_workload(w)
    yield s, d
    s.close()


def _block(n, p):
    rng = np.random.default_rng(p)
    return rng.standard_normal((n, p)), np.where(np.arange(p) % 3 == 1, 0.2, -0.1 - rng.uniform(0, 1, p))


@pytest.mark.parametrize("p", [1, 7, 8, 15, 16, 63, 64, 65, 511, 512, 1024])
def test_pointwise_apply(system, p):
    s, d = system
    print(f"[gpu] lp apply edges p={p}", flush=True)
    W = mlp.init_weights(7)
    W[5 * mlp.H:] = np.random.default_rng(8).standard_normal(mlp.H + 1) * 0.2
    W = W.astype(np.float32).astype(np.float64)
    s.lp_set_weights(W, NORM.astype(np.float32))
    G, lam = _block(d.n, p)
    P = s.lp_apply(lam, _dev(G)).cpu().numpy()
    dg = lambda A: np.asarray(d.csr(A).diagonal())
    ref = mlp.apply(W, NORM, dg(0.5 * d.L), dg(d.B), dg(d.H), lam, G)
    assert np.abs(P - ref).max() <= 2e-5 * np.abs(ref).max()


@pytest.mark.parametrize("p", [1, 3, 128, 129, 255, 256, 257])
def test_graph_gradient(system, p):
    s, d = system
    print(f"[gpu] gl gradient edges p={p}", flush=True)
    W = gnn.init_weights(4)
    rng = np.random.default_rng(104)
    W[5 * gnn.H:] = rng.standard_normal(2 * gnn.H + 2) * 0.15
    W[-1] += 0.5
    W = W.astype(np.float32).astype(np.float64)
    s.gl_set_weights(W, NORM)
    G, lam = _block(d.n, p)
    loss, grad = s.gl_loss_grad(lam, _dev(G))
    rl, rg = gnn.loss_grad(W, NORM, d.csr(0.5 * d.L), d.csr(d.B), np.asarray(d.csr(d.H).diagonal()), lam, G)
    assert abs(loss - rl) <= 2e-5 * abs(rl)
    assert np.abs(grad - rg).max() <= 2e-5 * np.abs(rg).max()
