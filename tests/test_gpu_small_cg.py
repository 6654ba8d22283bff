"""GPU: the inner CG of small blocks at the edges of its tiles (short last plan
blocks, fewer columns than a tile, broken last tiles, few iterations, columns
left as they are) against Jacobi-CG in extended precision on the same matrices."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _system(n):
    """Symmetric, diagonally dominant (condition number below 4 after the Jacobi
    scaling) L/2 and B of one banded pattern; H = L/2."""
    rng = np.random.default_rng(n)
    A = np.zeros((2, n, n))
    for r in range(n):
        for c in rng.choice(np.arange(r + 1, min(n, r + 40)), size=min(6, min(n, r + 40) - r - 1), replace=False):
            A[:, r, c] = A[:, c, r] = rng.uniform(-1, 1, 2)
    for k in range(2):
        A[k] += np.diag(2.0 * np.abs(A[k]).sum(1) + 0.5)
    rp, col = [0], []
    for r in range(n):
        c = np.flatnonzero(A[0][r])
        col.append(c)
        rp.append(rp[-1] + len(c))
    col = np.concatenate(col)
    rows = np.repeat(np.arange(n), np.diff(rp))
    return np.array(rp, dtype=np.int64), col.astype(np.int32), A[0][rows, col], A[1][rows, col], A


def _cg(T, g, m):
    J = 1.0 / np.diag(T)
    x, r = np.zeros_like(g), g.copy()
    z = J * r
    d, rz = z.copy(), r @ z
    for _ in range(m):
        q = T @ d
        a = rz / (d @ q)
        x, r = x + a * d, r - a * q
        z = J * r
        new = r @ z
        d, rz = z + new / rz * d, new
    return x


@pytest.mark.parametrize("m", [1, 2, 3, 10])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 300])
def test_small_block_cg(n, m):
    import torch
    from paper_2007_14228_amd import Solver
    rp, col, L, B, A = _system(n)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    s = Solver()
    s.csr_load(dev(rp), dev(col), dev(L), dev(B), dev(L))
    s.set_params(precond="paper", pcg_iters=m)
    wide = A.astype(np.longdouble)
    for p in (1, 2, 3, 15, 16, 17, 33):
        print(f"[gpu] small cg n={n} m={m} p={p}", flush=True)
        rng = np.random.default_rng(p)
        G = rng.standard_normal((n, p))
        lam = np.where(np.arange(p) % 4 == 2, 0.3, -rng.uniform(0.1, 3.0, p))
        P = s.precondition(lam, dev(G)).cpu().numpy()
        for c in range(p):
            if lam[c] >= 0:
                assert np.array_equal(P[:, c], G[:, c])
                continue
            # past the matrix's dimension nothing is left to iterate on
            ref = _cg(wide[0] - np.longdouble(lam[c]) * wide[1], G[:, c].astype(np.longdouble), min(m, n))
            # ten steps of rows of a dozen products each: a few hundred roundings of 2^-53, condition number 4
            assert np.abs(P[:, c] - ref).max() <= 2e-13 * np.abs(ref).max(), (c, p)
    s.close()


@pytest.mark.parametrize("mode", ["auto", "halo", "gather"])
def test_iterations_past_the_solution_change_nothing(mode):
    """Diagonal matrices: Jacobi-CG has the solution after one step, and the
    steps after it must leave it alone, in every form of the iteration."""
    import torch
    from paper_2007_14228_amd import Solver
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for n, p in ((1, 6), (2, 5), (200, 8), (3000, 900)):
        print(f"[gpu] cg past the solution {mode} n={n} p={p}", flush=True)
        rng = np.random.default_rng(n)
        L, B = rng.uniform(1, 2, n), rng.uniform(1, 2, n)
        rp, col = np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32)
        s = Solver()
        s.csr_load(dev(rp), dev(col), dev(L), dev(B), dev(L))
        s.set_params(precond="paper", pcg_iters=40, spmm_mode=mode)
        G, lam = rng.standard_normal((n, p)), -rng.uniform(0.1, 3.0, p)
        P = s.precondition(lam, dev(G)).cpu().numpy()
        ref = G / (L[:, None] - lam * B[:, None])
        # the quotient's few roundings, twice over for the steps' remainders
        assert np.abs(P - ref).max() <= 1e-14 * np.abs(ref).max()
        s.close()


@pytest.mark.parametrize("n", [250 * 64, 257 * 64, 1536 * 64, 1537 * 64 + 1])
def test_partial_sums_on_both_sides_of_their_groupings(n):
    """Three iterations on tridiagonal matrices, with as many plan blocks as the
    dots' partials change their way to the sum at, against the same in FP64."""
    import scipy.sparse as sp
    import torch
    from paper_2007_14228_amd import Solver
    print(f"[gpu] cg partials n={n}", flush=True)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    rng = np.random.default_rng(n)
    mats = []
    for _ in range(2):
        o = rng.uniform(-1, 1, n - 1)
        mats.append(sp.diags([o, rng.uniform(3, 4, n), o], [-1, 0, 1]).tocsr())
    L, B = mats
    s = Solver()
    s.csr_load(dev(L.indptr.astype(np.int64)), dev(L.indices.astype(np.int32)), dev(L.data), dev(B.data), dev(L.data))
    s.set_params(precond="paper", pcg_iters=3, spmm_mode="halo")
    p = 12
    G, lam = rng.standard_normal((n, p)), -rng.uniform(0.1, 3.0, p)
    P = s.precondition(lam, dev(G)).cpu().numpy()
    for c in range(p):
        ref = _cg_sparse(L - lam[c] * B, G[:, c], 3)
        # sums of 1e5 terms by trees and a few dozen roundings a value, condition number below 7
        assert np.abs(P[:, c] - ref).max() <= 1e-13 * np.abs(ref).max(), c
    s.close()


def _cg_sparse(T, g, m):
    J = 1.0 / T.diagonal()
    x, r = np.zeros_like(g), g.copy()
    d = J * r
    rz = r @ d
    for _ in range(m):
        q = T @ d
        a = rz / (d @ q)
        x, r = x + a * d, r - a * q
        z = J * r
        new = r @ z
        d, rz = z + new / rz * d, new
    return x
