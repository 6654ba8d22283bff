"""GPU: rounding of the FP64 Gram at the widths where its kernels and its column
sums change (p = 45 and 46: 64 columns a block from 4096 sums on; 64 and 65)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [16, 45, 46, 64, 65, 128])
def test_gram_rounding(p):
    import torch
    from paper_2007_14228_amd import Solver
    n = 120_000
    print(f"[gpu] gram rounding p={p}", flush=True)
    eye = [torch.arange(n + 1, dtype=torch.int64, device="cuda"), torch.arange(n, dtype=torch.int32, device="cuda")]
    one = torch.ones(n, dtype=torch.float64, device="cuda")
    s = Solver()
    s.csr_load(*eye, one, one)
    diag, off = [], []
    for seed in range(4):
        g = torch.Generator(device="cuda").manual_seed(seed)
        X, E = (torch.randn(n, p, dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
        HX, BX = -2.0 * X + 0.3 * E, 0.02 * X + 0.002 * E
        S, L0 = s.gram(X, HX, BX)
        Xl = X[:, :16].cpu().numpy().astype(np.longdouble)
        for Y, G in ((BX, S), (HX, L0)):
            Yl = Y[:, :16].cpu().numpy().astype(np.longdouble)
            ref = np.stack([(Xl[:, i:i + 1] * Yl).sum(0) for i in range(16)])
            d = np.sqrt(np.abs(np.diag(ref))).astype(float)
            e = (G[:16, :16] - ref).astype(float) / (d[:, None] * d)
            diag.append(np.diag(e))
            off.append(e[~np.eye(16, dtype=bool)])
    rms = lambda v: float(np.sqrt(np.mean(np.square(np.concatenate(v)))))
    s.close()
    # On the diagonal the sum's own rounding (2^-53 / sqrt 3 = 0.6e-16 at worst) and
    # as much again for the way there; beside it the partial sums are random walks of
    # sqrt(rows) terms, a thousandth of that, in chains of up to a few dozen fours of rows
    assert rms(diag) <= 0.9e-16, rms(diag)
    assert rms(off) <= 1.8e-18, rms(off)
