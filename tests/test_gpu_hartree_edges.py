"""GPU: the Hartree solve at the edges of its kernel's tiles (fewer rows than a
block, short last blocks, several blocks a workgroup, rows of up to 16, 32 and
64 entries): the potential's residual against the matrix and the density that
the library itself reports."""
import math

import numpy as np
import pytest
import scipy.sparse as sp
from scipy.spatial import Delaunay

import workloads as wl
from oracle import fem

pytestmark = pytest.mark.gpu


def _cube(cells):
    ax = wl.uniform_axis(-4.0, 4.0, cells)
    return wl.kuhn_mesh(ax, ax, ax)


def _star(spokes):
    """A node in the middle of a sphere of `spokes` nodes, in a box: one long row."""
    k = np.arange(spokes) + 0.5
    z, phi = 1.0 - 2.0 * k / spokes, math.pi * (1.0 + math.sqrt(5.0)) * k
    r = np.sqrt(1.0 - z * z)
    g = np.array([(x, y, q) for x in (-3.0, 0.1, 3.0) for y in (-3.0, 0.2, 3.0) for q in (-3.0, 0.3, 3.0)])
    g = g[np.abs(g).max(1) > 1.0]
    xyz = np.concatenate([[[0.0, 0.0, 0.0]], np.stack([r * np.cos(phi), r * np.sin(phi), z], 1), g])
    tets = Delaunay(xyz).simplices.astype(np.int32)
    e = xyz[tets[:, 1:]] - xyz[tets[:, :1]]
    det = np.linalg.det(e)
    tets = tets[np.abs(det) > 1e-9]
    flip = np.linalg.det(xyz[tets[:, 1:]] - xyz[tets[:, :1]]) < 0
    tets[flip] = tets[flip][:, [0, 2, 1, 3]]
    return wl.Mesh(xyz=xyz, tets=tets, dirichlet=(np.abs(xyz).max(1) > 2.9).astype(np.uint8), cells=())


MESHES = {
    "one row": lambda: _cube(2), "27 rows": lambda: _cube(4), "64 rows": lambda: _cube(5),
    "125 rows": lambda: _cube(6), "two blocks a workgroup": lambda: _cube(42),
    "32 entries": lambda: _star(24), "64 entries": lambda: _star(50),
}


@pytest.mark.parametrize("graphs", [0, 1])
@pytest.mark.parametrize("which", list(MESHES))
def test_hartree_potential_at_tile_edges(which, graphs):
    import torch
    from paper_2007_14228_amd import Solver
    mesh = MESHES[which]()
    w = wl.Workload("edge", mesh, np.array([2.0]), np.array([[0.31, 0.17, 0.23]]), p=1, beta=1.0, scf=True, seed=0)
    print(f"[gpu] hartree edges {which} n={mesh.n_dofs} graphs={graphs}", flush=True)
    s = Solver()
    s.load_workload(w)
    rtol = 1e-10
    s.set_params(beta=w.beta, precond="paper", scf=1, use_graphs=graphs, poisson_rtol=rtol, poisson_max_iter=20000)
    m = s.csr_get()
    n = len(m["row_ptr"]) - 1
    longest = int(np.diff(m["row_ptr"]).max())
    if which.endswith("entries"):
        lo, hi = (17, 32) if which == "32 entries" else (33, 64)
        assert lo <= longest <= hi
    X = np.random.default_rng(n).standard_normal((n, 1))
    for _ in range(2):                                     # the second solve starts from the first one's potential
        got = s.build_hamiltonian(torch.from_numpy(X).cuda())
        rho, U = got["rho"].cpu().numpy(), got["U"].cpu().numpy()
        d = fem.discretize(mesh, w.Z, w.R)
        loc = (d.vol[:, None] / 4.0 * rho) @ fem.BARY
        dv = d.dof[d.tets].ravel()
        rhs = 4.0 * math.pi * np.bincount(dv[dv >= 0], weights=loc.ravel()[dv >= 0], minlength=n)
        L = sp.csr_matrix((m["L"], m["col"], m["row_ptr"]), shape=(n, n))
        # the solver's own bound, and the rounding of r = rhs - L U over its updates
        slack = 1e-12 * (np.linalg.norm(rhs) + np.linalg.norm(abs(L) @ np.abs(U)))
        assert np.linalg.norm(rhs - L @ U) <= 1.001 * rtol * np.linalg.norm(rhs) + slack
        X *= 1.1
    s.close()


@pytest.mark.parametrize("graphs", [0, 1])
def test_hartree_iteration_limit_is_kept(graphs):
    """Too few iterations are an error, whatever was queued ahead; the next solve
    goes on from the potential that they left and reaches its bound."""
    import torch
    from paper_2007_14228_amd import Solver
    mesh = _cube(20)
    w = wl.Workload("edge", mesh, np.array([2.0]), np.array([[0.31, 0.17, 0.23]]), p=1, beta=1.0, scf=True, seed=0)
    print(f"[gpu] hartree limit graphs={graphs}", flush=True)
    s = Solver()
    s.load_workload(w)
    X = torch.from_numpy(np.random.default_rng(3).standard_normal((mesh.n_dofs, 1))).cuda()
    prm = dict(beta=w.beta, precond="paper", scf=1, use_graphs=graphs, poisson_rtol=1e-11)
    for limit in (1, 10, 11, 20):                          # one ten, one, two, two: none is enough
        s.set_params(poisson_max_iter=limit, **prm)
        with pytest.raises(RuntimeError, match="Hartree CG"):
            s.build_hamiltonian(X)
    s.set_params(poisson_max_iter=5000, **prm)
    a = s.build_hamiltonian(X)["U"].cpu().numpy()
    b = s.build_hamiltonian(X)["U"].cpu().numpy()          # starts at the solution: nothing to do
    assert np.isfinite(a).all() and np.array_equal(a, b)
    s.close()
