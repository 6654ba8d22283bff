"""GPU: the LDS-halo products at the edges of their tiles (column slices,
rounds of sixteen row entries, unaligned blocks, short last blocks) against
dense FP64 products of the same matrices."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _system(n, longest):
    """Rows of 1 to `longest` entries in a band, with their diagonal; H, B, L/2."""
    rng = np.random.default_rng(longest)
    rows = []
    for r in range(n):
        lo, hi = max(0, r - 40), min(n, r + 41)
        want = 1 + (r * 7) % longest
        cols = rng.permutation(np.arange(lo, hi))[:want]
        cols[0] = r if r not in cols else cols[0]
        rows.append(np.sort(np.unique(cols)))
    rp = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int64)
    col = np.concatenate(rows).astype(np.int32)
    vals = [rng.standard_normal(col.size) for _ in range(3)]
    dense = []
    for v in vals:
        A = np.zeros((n, n))
        A[np.repeat(np.arange(n), np.diff(rp)), col] = v
        dense.append(A)
    return rp, col, vals, dense


@pytest.mark.parametrize("longest", [15, 16, 17, 33, 64])
@pytest.mark.parametrize("n", [63, 65, 700])
def test_halo_products_at_tile_edges(n, longest):
    import torch

    from paper_2007_14228_amd import Solver
    rp, col, vals, (H, B, L) = _system(n, longest)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    s = Solver()
    s.csr_load(dev(rp), dev(col), *map(dev, vals))
    s.set_params(precond="paper", spmm_mode="halo")
    rng = np.random.default_rng(n)
    for dt, eps in ((np.float64, 2.0 ** -53), (np.float32, 2.0 ** -24)):
        for p in (1, 4, 31, 32, 33, 64, 66, 131):
            for shift in (0, 1):                       # 1: the block starts one element past its allocation
                print(f"[gpu] halo edges n={n} longest={longest} {dt.__name__} p={p} offset={shift}", flush=True)
                flat = rng.standard_normal(n * p + shift).astype(dt)
                X = dev(flat)[shift:].view(n, p)
                Xd = flat[shift:].reshape(n, p).astype(np.float64)
                lam = rng.standard_normal(p)
                HX, BX = s.spmm_ex(X, "dual")
                Q = s.spmm_ex(X, "shift", lam)
                # rounding of the values and of sums of at most 64 products, for each of the two matrices
                bound = lambda A: 70 * eps * (np.abs(A) @ np.abs(Xd)) + 1e-300
                assert np.all(np.abs(HX.cpu().numpy() - H @ Xd) <= bound(H))
                assert np.all(np.abs(BX.cpu().numpy() - B @ Xd) <= bound(B))
                ref = np.where(lam < 0, L @ Xd - lam * (B @ Xd), 0.0)
                assert np.all(np.abs(Q.cpu().numpy() - ref) <= 2 * (bound(L) + np.abs(lam) * bound(B)))


def test_a_non_finite_row_reaches_its_neighbours_only():
    import torch

    from paper_2007_14228_amd import Solver
    n, p = 300, 40
    rp, col, vals, (H, B, L) = _system(n, 20)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    s = Solver()
    s.csr_load(dev(rp), dev(col), *map(dev, vals))
    s.set_params(precond="paper", spmm_mode="halo")
    X = np.random.default_rng(1).standard_normal((n, p))
    X[150] = np.inf
    X[151] = np.nan
    touched = (H[:, 150] != 0) | (H[:, 151] != 0)
    for Y in s.spmm(dev(X)):
        finite = np.isfinite(Y.cpu().numpy())
        assert not finite[touched].any() and finite[~touched].all()
