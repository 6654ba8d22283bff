"""GPU: the Gram at the edges of its tiles (16-column tiles, rows per wave and
split, the switch of kernels at p = 64) against FP64 products on the host."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 17, 513, 5000])
def test_gram_at_tile_edges(n):
    import torch

    from paper_2007_14228_amd import Solver
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    s = Solver()
    one = np.ones(n)
    s.csr_load(dev(np.arange(n + 1)), dev(np.arange(n, dtype=np.int32)), *(dev(one) for _ in range(3)))
    rng = np.random.default_rng(n)
    for p in (1, 15, 16, 17, 31, 33, 47, 48, 49, 63, 64, 65, 129):
        print(f"[gpu] gram edges n={n} p={p}", flush=True)
        X, H, B = (rng.standard_normal((n, p)) for _ in range(3))
        S, L0 = s.gram(dev(X), dev(H), dev(B))
        S2, L2 = s.gram(dev(X), dev(H), dev(B))
        assert np.array_equal(S, S2) and np.array_equal(L0, L2)      # fixed summation order
        eps = 2.0 ** -53
        assert np.all(np.abs(S - X.T @ B) <= 2 * (n + 4) * eps * (np.abs(X).T @ np.abs(B)))
        assert np.all(np.abs(L0 - X.T @ H) <= 2 * (n + 4) * eps * (np.abs(X).T @ np.abs(H)))
