"""The work that a user of the solver has it do, as cases that can be timed.

A case is one call (or one short sequence of calls) through `Solver`:

  step     set_x0 and a few iterations of Algorithm PCAL from a start block,
           then get_x: the whole call, as linear problem (fixed H) in either
           block precision or as Kohn-Sham SCF
  product  the dual product H X, B X, or the shifted product (L/2 - lam B) X
  gram     S = X^T B X and Lambda0 = X^T H X
  solve    the paper preconditioner T^-1 G (ten Jacobi-CG steps a column)
  density  two successive updates of density, potential and H(X), as an SCF
           loop makes them (the second is warm-started by the first)
  learned  the pointwise learned preconditioner, inference
  train    loss and parameter gradient of the graph preconditioner

Systems: "kuhn" is a graded tensor grid of tetrahedra with nuclei, assembled
by the library (interior rows of 15 entries); "irregular" is a CSR matrix
given as such, with the row lengths of a Delaunay mesh (7 to 27 entries).
Both number their nodes along the Z-order curve.  Nuclei, blocks, shifts,
weights (and the irregular pattern) come from the seed.

`exact` evaluates the same definitions in 64 bits with plain torch: its own
assembly, products by gathered rows, textbook CG.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2007_14228_amd import Solver

DEV = "cuda"
HALF = 10.0          # the box is [-HALF, HALF]^3
F64 = torch.float64


# ----------------------------------------------------------------------------
# The cases
# ----------------------------------------------------------------------------

def listed():
    return [
        # the smallest whole call: one nucleus on a uniform-sized grid of 16^3
        # cells, p = 4; launches, host algebra and synchronizations count
        dict(name="step_small", kind="step", system="kuhn", cells=16, p=4, precision="f64", steps=5, scf=0),
        # the mixed-precision run's first phase: the same in FP32 blocks
        dict(name="step_f32", kind="step", system="kuhn", cells=81, p=128, precision="f32", steps=3, scf=0),
        # many orbitals (96 nuclei), where the O(n p^2) contractions weigh most
        dict(name="step_wide", kind="step", system="kuhn", cells=49, p=512, precision="f64", steps=2, scf=0),
        # a small molecule's SCF iterations (p = 11: odd width, unaligned rows)
        dict(name="step_scf", kind="step", system="kuhn", cells=41, p=11, precision="f64", steps=2, scf=1),
        # the dual product at the headline width
        dict(name="product_dual", kind="product", system="kuhn", cells=81, p=128, precision="f64", op="dual"),
        # the shifted product of the FP32 phase, at a width that is no multiple of 128
        dict(name="product_shift_f32", kind="product", system="kuhn", cells=81, p=160, precision="f32", op="shift"),
        # the Gram of a medium block (no power of two)
        dict(name="gram_48", kind="gram", system="kuhn", cells=59, p=48),
        # the paper preconditioner on a matrix with irregular rows, a narrow block
        dict(name="solve_irregular", kind="solve", system="irregular", cells=50, p=16),
        # the SCF density update at the size of a 4-nucleus all-electron mesh
        dict(name="density", kind="density", system="kuhn", cells=59, p=11),
        # the learned preconditioner's inference
        dict(name="learned", kind="learned", system="kuhn", cells=59, p=64),
        # one training step's gradient of the graph preconditioner
        dict(name="train", kind="train", system="kuhn", cells=38, p=16),
        # the headline work: FP64 iterations of a 24-nucleus cluster, p = 128,
        # on a grid whose blocks (1 GB) are far beyond every cache
        dict(name="step_f64", kind="step", system="kuhn", cells=101, p=128, precision="f64", steps=3, scf=0),
    ]


# draw: kind -> (weight, cells from, cells to, p from, p to, largest n p)
RANGES = {
    "step": (5, 12, 80, 2, 512, 3.0e7),
    "product": (4, 12, 80, 3, 512, 8.0e7),
    "gram": (3, 12, 80, 2, 512, 6.0e7),
    "solve": (4, 12, 70, 2, 384, 4.0e7),
    "density": (2, 12, 60, 2, 48, 4.0e6),
    "learned": (1, 12, 70, 2, 256, 4.0e7),
    "train": (1, 10, 45, 2, 64, 2.0e6),
}


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kinds = sorted(RANGES)
    kind = rng.choices(kinds, weights=[RANGES[k][0] for k in kinds])[0]
    _, c0, c1, p0, p1, most = RANGES[kind]
    cells = _log_int(rng, c0, c1)
    p = _log_int(rng, p0, p1)
    if rng.random() < 0.5 and p > 16:
        p = (p + 4) // 8 * 8                # half of the wider blocks at multiples of 8, the others as they fall
    n = (cells - 1) ** 3
    p = max(1, min(p, n // 8, int(most / n)))
    case = dict(kind=kind, system="kuhn", cells=cells, p=p)
    if kind in ("product", "solve") and rng.random() < 0.4:
        case["system"] = "irregular"
    if kind == "product":
        case["precision"] = rng.choice(["f64", "f32"])
        case["op"] = rng.choice(["dual", "shift"])
    if kind == "step":
        case["scf"] = 1 if p <= 24 and n <= 80_000 and rng.random() < 0.4 else 0
        case["precision"] = "f64" if case["scf"] else rng.choice(["f64", "f64", "f32"])
        case["steps"] = rng.randint(2, 3)
    return case


# ----------------------------------------------------------------------------
# Systems
# ----------------------------------------------------------------------------

def _morton(i, j, k):
    code = np.zeros(i.shape, dtype=np.int64)
    for b in range(8):
        for d, a in enumerate((i, j, k)):
            code |= ((a >> b) & 1) << (3 * b + d)
    return code


@functools.lru_cache(maxsize=2)
def _grid(cells):
    """Graded tensor grid of tetrahedra on [-HALF, HALF]^3, spacing finer
    towards the middle: xyz [N, 3], tets [6 cells^3, 4], dirichlet [N]; nodes
    in Z-order, tetrahedra by their lowest node.  (Geometry only, the same for
    every seed; kept so that several inputs of one size share it.)"""
    t = np.linspace(-1.0, 1.0, cells + 1)
    ax = HALF * np.sinh(2.0 * t) / math.sinh(2.0)
    m = cells + 1
    i, j, k = (a.ravel().astype(np.int64) for a in np.meshgrid(*[np.arange(m)] * 3, indexing="ij"))
    order = np.argsort(_morton(i, j, k), kind="stable")
    rank = np.empty_like(order)
    rank[order] = np.arange(order.size)
    i, j, k = i[order], j[order], k[order]
    xyz = np.stack([ax[i], ax[j], ax[k]], axis=1)
    edge = np.zeros(order.size, dtype=np.uint8)
    for a in (i, j, k):
        edge |= (a == 0) | (a == cells)
    low = (i < cells) & (j < cells) & (k < cells)
    ci, cj, ck = i[low], j[low], k[low]
    tets = np.empty((ci.size, 6, 4), dtype=np.int32)
    for q, axes in enumerate(((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0))):
        at = [ci.copy(), cj.copy(), ck.copy()]
        tets[:, q, 0] = rank[(at[0] * m + at[1]) * m + at[2]]
        for v, a in enumerate(axes):
            at[a] += 1
            tets[:, q, v + 1] = rank[(at[0] * m + at[1]) * m + at[2]]
    tets = tets.reshape(-1, 4)
    tets = np.ascontiguousarray(tets[np.argsort(tets.min(axis=1), kind="stable")])
    return xyz, tets, edge


def _nuclei(case, seed):
    """Charges (in turn 8, 1, 7, 6) and positions: for SCF and density work the
    neutral cluster of p orbitals (4 nuclei for 11), else 3 nuclei for 16."""
    neutral = case["kind"] == "density" or case.get("scf")
    count = max(1, math.ceil(case["p"] * (4 / 11 if neutral else 3 / 16)))
    reach = min(6.0, 3.0 * (count / 4.0) ** (1.0 / 3.0))
    Z = np.array([(8.0, 1.0, 7.0, 6.0)[j % 4] for j in range(count)])
    return Z, np.random.default_rng(seed).uniform(-reach, reach, size=(count, 3))


def _irregular(cells, seed):
    """Symmetric CSR matrices (H, B, L/2) on (cells - 1)^3 nodes in Z-order: each
    node couples to its 6 face neighbours and to a random part of the 12 edge
    and 8 corner neighbours, as on a Delaunay mesh."""
    m = cells - 1
    g = torch.Generator(device=DEV).manual_seed(seed)
    i, j, k = (a.ravel().astype(np.int64) for a in np.meshgrid(*[np.arange(m)] * 3, indexing="ij"))
    order = np.argsort(_morton(i, j, k), kind="stable")
    rank = np.empty_like(order)
    rank[order] = np.arange(order.size)
    i, j, k = (torch.from_numpy(a[order]).to(DEV) for a in (i, j, k))
    rank = torch.from_numpy(rank).to(DEV)
    n = m ** 3
    row = torch.arange(n, device=DEV)
    keep_of = {1: 1.1, 2: 0.6, 3: 0.4}
    rows, cols, lv, bv = [], [], [], []
    diag_l = torch.full((n,), 0.05, dtype=F64, device=DEV)
    diag_b = torch.full((n,), 0.02, dtype=F64, device=DEV)
    for d in [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1) if (a, b, c) > (0, 0, 0)]:
        ii, jj, kk = i + d[0], j + d[1], k + d[2]
        ok = (ii >= 0) & (ii < m) & (jj >= 0) & (jj < m) & (kk >= 0) & (kk < m)
        ok &= torch.rand(n, device=DEV, generator=g) < keep_of[sum(map(abs, d))]
        w = (0.5 + torch.rand(n, dtype=F64, device=DEV, generator=g))[ok]
        b = 0.02 * (0.5 + torch.rand(n, dtype=F64, device=DEV, generator=g))[ok]
        r, c = row[ok], rank[((ii * m + jj) * m + kk)[ok]]
        rows += [r, c]
        cols += [c, r]
        lv += [-w, -w]
        bv += [b, b]
        for a in (r, c):
            diag_l.index_add_(0, a, w)
            diag_b.index_add_(0, a, b)
    rows, cols = torch.cat(rows + [row]), torch.cat(cols + [row])
    lv, bv = torch.cat(lv + [diag_l]), torch.cat(bv + [diag_b])
    at = torch.argsort(rows * n + cols)
    rows, cols, lv, bv = rows[at], cols[at], lv[at].contiguous(), bv[at].contiguous()
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    pot = -4.0 * torch.rand(n, dtype=F64, device=DEV, generator=g)
    hv = lv + 0.5 * (pot[rows] + pot[cols]) * bv
    return rp, cols.to(torch.int32), hv, bv, lv


def _solver(case, seed):
    s = Solver()
    if case["system"] == "irregular":
        s.csr_load(*_irregular(case["cells"], seed))
    else:
        xyz, tets, edge = _grid(case["cells"])
        s.mesh_load(xyz, tets, edge)
        s.nuclei_set(*_nuclei(case, seed))
        s.assemble()
    return s


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------

def _block(case, seed, which=0):
    g = torch.Generator(device=DEV).manual_seed(1000 * seed + which)
    return torch.randn(((case["cells"] - 1) ** 3, case["p"]), dtype=F64, device=DEV, generator=g)


def _shifts(case, seed):
    """Multiplier diagonals as an iteration meets them once the orbitals are bound: negative."""
    r = np.random.default_rng(seed + 7)
    return -np.exp(r.uniform(math.log(0.05), math.log(20.0), size=case["p"]))


def _orbitals(case, seed, which=0):
    """A start block as atoms suggest it: in each column an exponential around a
    nucleus, times a wave (bound, so the preconditioner works from the start;
    far from linearly dependent)."""
    xyz, _, edge = _grid(case["cells"])
    x = torch.from_numpy(xyz[edge == 0]).to(DEV)
    Z, R = _nuclei(case, seed)
    r = np.random.default_rng(seed + 31 * which + 5)
    out = torch.empty((x.shape[0], case["p"]), dtype=F64, device=DEV)
    for c in range(case["p"]):
        j = c % len(R)
        a, wave, phase = r.uniform(0.5, max(1.0, 0.6 * Z[j])), r.uniform(-2.0, 2.0, 3), r.uniform(0.0, 2.0 * math.pi)
        d = x - torch.from_numpy(R[j]).to(DEV)
        out[:, c] = (a ** 3 / math.pi) ** 0.5 * torch.exp(-a * d.norm(dim=1)) * torch.cos(d @ torch.from_numpy(wave).to(DEV) + phase)
    return out


def _weights(seed, count):
    """A network of small random weights and plausible standardization."""
    r = np.random.default_rng(seed + 3)
    w = (0.3 * r.standard_normal(count)).astype(np.float32)
    return w, np.array([-1.0, -4.0, -2.0, 0.0, 2.0, 2.0, 4.0, 1.0], dtype=np.float32)


PARAMS = dict(tol=1e-30, precond="paper", pcg_iters=10)


def prepare(case, seed):
    kind = case["kind"]
    state = dict(case=case, s=_solver(case, seed))
    s = state["s"]
    if kind == "step":
        s.set_params(**PARAMS, scf=case["scf"], precision=case["precision"], max_iter=case["steps"])
        state["X"] = _orbitals(case, seed)
    else:
        s.set_params(**PARAMS)
    if kind == "product":
        state["X"] = _block(case, seed).to(F64 if case["precision"] == "f64" else torch.float32)
        state["lam"] = _shifts(case, seed)
    elif kind == "gram":
        X = _block(case, seed)
        state["blocks"] = X, -2.0 * X + 3.0 * _block(case, seed, 1), 0.02 * X + 0.01 * _block(case, seed, 2)
    elif kind in ("solve", "learned", "train"):
        state["G"] = _block(case, seed)
        state["lam"] = _shifts(case, seed)
        if kind == "learned":
            s.lp_set_weights(*_weights(seed, 193))
        elif kind == "train":
            s.gl_set_weights(*_weights(seed, 226))
    elif kind == "density":
        a, b = _orbitals(case, seed), _orbitals(case, seed, 1)
        state["X"] = a, 0.95 * a + 0.1 * b
    return state


# ----------------------------------------------------------------------------
# One pass
# ----------------------------------------------------------------------------

STATS = ("energy", "kkt", "fea", "rel", "eta")


def run(state):
    case, s = state["case"], state["s"]
    kind = case["kind"]
    if kind == "step":
        s.set_x0(state["X"])
        log, _, _ = s.step(case["steps"] + 1)      # stops at max_iter, with the last iterate evaluated
        X = s.get_x()
        stats = np.array([[it[f] for f in STATS] for it in log])
        if case["precision"] == "f32":      # FP32 iterates: returned in the precision that they have
            return dict(X=X.float(), stats=stats.astype(np.float32))
        return dict(X=X, stats=stats)
    if kind == "product":
        return s.spmm_ex(state["X"], case["op"], state["lam"] if case["op"] == "shift" else None)
    if kind == "gram":
        return s.gram(*state["blocks"])
    if kind == "solve":
        return s.precondition(state["lam"], state["G"])
    if kind == "density":
        return [s.build_hamiltonian(X) for X in state["X"]]
    if kind == "learned":
        return s.lp_apply(state["lam"], state["G"])
    return s.gl_loss_grad(state["lam"], state["G"])


def work(case):
    """What a pass cannot do without: its inputs read once and its outputs
    written once; for the iterative calls, each product of an inner step
    reading and writing a block, and each recurrence its operands, since no
    cache holds a block from one step to the next."""
    n, p, kind = (case["cells"] - 1) ** 3, case["p"], case["kind"]
    w = 4 if case.get("precision") == "f32" else 8
    nnz = 15 * n
    mat = nnz * (2 * w + 4)
    blk = n * p * w
    tets = 6 * case["cells"] ** 3
    cg = 600 * (12 * nnz + 9 * 8 * n)       # one Hartree solve: a product and two recurrences a step
    dens = 4 * tets * p * w + 3 * 32 * tets + 4 * 8 * nnz
    if kind == "product":
        one = case["op"] == "shift"
        return dict(bytes=(2 if one else 3) * blk + mat, flops=4.0 * nnz * p)
    if kind == "gram":
        return dict(bytes=3 * blk, flops=4.0 * n * p * p)
    if kind == "solve":
        return dict(bytes=10 * (6 * blk + mat) + 2 * blk, flops=10.0 * (4 * nnz + 10 * n) * p)
    if kind == "density":
        return dict(bytes=2 * (dens + cg), flops=2 * (4.0 * tets * p * 10 + 600.0 * 2 * nnz))
    if kind == "learned":
        return dict(bytes=3 * blk, flops=330.0 * n * p)
    if kind == "train":
        return dict(bytes=3 * (2 * blk + mat) + 10 * blk, flops=1500.0 * n * p)
    it = 3 * blk + mat + 3 * blk + 4 * blk + 8 * blk + 10 * (6 * blk + mat)
    return dict(bytes=case["steps"] * (it + case["scf"] * (dens + cg)) + 6 * blk,
                flops=case["steps"] * (8.0 * n * p * p + 48.0 * nnz * p) + 4.0 * n * p * p)


# ----------------------------------------------------------------------------
# The same in 64 bits
# ----------------------------------------------------------------------------

QA = (5.0 + 3.0 * math.sqrt(5.0)) / 20.0
QB = (5.0 - math.sqrt(5.0)) / 20.0


class _System:
    """L/2, B and H as rows padded to one length (col, values [n, width])."""

    def __init__(self, case, seed):
        if case["system"] == "irregular":
            rp, col, hv, bv, lv = _irregular(case["cells"], seed)
            self.n = rp.numel() - 1
            self.rows = torch.repeat_interleave(torch.arange(self.n, device=DEV), rp[1:] - rp[:-1])
            self.cols, self.first = col.long(), rp
            self._pad()
            self.Lh, self.B, self.H = (self._ell(v) for v in (lv, bv, hv))
        else:
            self._assemble(case, seed)
        own = self.col == torch.arange(self.n, device=DEV)[:, None]
        self.lhd, self.bd = ((v * own).sum(1) for v in (self.Lh, self.B))
        self.own = own

    def _pad(self):
        at = torch.arange(self.rows.numel(), device=DEV) - self.first[self.rows]
        width = int(at.max()) + 1
        self.at = at
        self.col = torch.full((self.n, width), -1, device=DEV)      # -1: padding (its values are zero)
        self.col[self.rows, at] = self.cols

    def _ell(self, v):
        out = torch.zeros(self.col.shape, dtype=F64, device=DEV)
        out[self.rows, self.at] = v
        return out

    def _assemble(self, case, seed):
        xyz, tets, edge = (torch.from_numpy(a).to(DEV) for a in _grid(case["cells"]))
        Z, R = (torch.from_numpy(a).to(DEV) for a in _nuclei(case, seed))
        dof = torch.cumsum((edge == 0).long(), 0) - 1
        dof[edge != 0] = -1
        self.n = n = int(dof.max()) + 1
        v = xyz[tets.long()]
        e1, e2, e3 = (v[:, a] - v[:, 0] for a in (1, 2, 3))
        det = (e1 * torch.linalg.cross(e2, e3)).sum(1, keepdim=True)
        vol = det[:, 0].abs() / 6.0
        g = torch.stack([torch.linalg.cross(e2, e3), torch.linalg.cross(e3, e1), torch.linalg.cross(e1, e2)], 2)
        g = g / det[:, :, None]                         # [t, d, a]: gradients of the barycentric coordinates 1 to 3
        g = torch.cat([-g.sum(2, keepdim=True), g], 2)
        self.vol, self.dt = vol, dof[tets.long()]
        bary = torch.full((4, 4), QB, dtype=F64, device=DEV).fill_diagonal_(QA)
        self.bary = bary
        xq = torch.einsum("qa,tad->tqd", bary, v)
        vext = torch.zeros(xq.shape[:2], dtype=F64, device=DEV)
        for z, r in zip(Z, R):
            vext -= z / (xq - r).norm(dim=2)
        self.vext = vext
        a, b = torch.meshgrid(torch.arange(4, device=DEV), torch.arange(4, device=DEV), indexing="ij")
        self.pair = a.ravel(), b.ravel()
        i, j = self.dt[:, self.pair[0]], self.dt[:, self.pair[1]]
        self.inner = ((i >= 0) & (j >= 0)).ravel()
        uniq, self.where = torch.unique((i * n + j).ravel()[self.inner], return_inverse=True)
        self.rows, self.cols = uniq // n, uniq % n
        self.first = torch.searchsorted(self.rows, torch.arange(n + 1, device=DEV))
        self._pad()
        stiff = vol[:, None] * sum(g[:, d][:, self.pair[0]] * g[:, d][:, self.pair[1]] for d in range(3))
        mass = vol[:, None] * (1.0 + (self.pair[0] == self.pair[1]).double()) / 20.0
        self.Lh, self.B = 0.5 * self._scatter(stiff), self._scatter(mass)
        self.H = self.Lh + self._potential(vext)

    def _scatter(self, loc):
        out = torch.zeros(self.rows.numel(), dtype=F64, device=DEV)
        out.index_add_(0, self.where, loc.ravel()[self.inner])
        return self._ell(out)

    def _potential(self, vq):
        w = 0.25 * self.vol[:, None] * vq
        return self._scatter(w @ (self.bary[:, self.pair[0]] * self.bary[:, self.pair[1]]))

    def times(self, val, X, val2=None):
        """val X (and val2 X)."""
        col = self.col.clamp(min=0)
        Y = torch.zeros_like(X)
        Y2 = torch.zeros_like(X) if val2 is not None else None
        for j in range(col.shape[1]):
            x = X[col[:, j]]
            Y += val[:, j, None] * x
            if val2 is not None:
                Y2 += val2[:, j, None] * x
        return Y if val2 is None else (Y, Y2)

    def shifted(self, lam, X):
        a, b = self.times(self.Lh, X, self.B)
        return a - lam * b

    def hd(self):
        return (self.H * self.own).sum(1)

    def solve(self, lam, G, steps=10):
        """Jacobi-CG on (L/2 - lam B) x = g from zero; columns with lam >= 0 are copied."""
        on = lam < 0
        P = G.clone()
        if not bool(on.any()):
            return P
        l, r = lam[on], G[:, on].clone()
        J = 1.0 / (self.lhd[:, None] - l * self.bd[:, None])
        x, z = torch.zeros_like(r), r * J
        d, rz = z.clone(), (r * z).sum(0)
        for _ in range(steps):
            q = self.shifted(l, d)
            alpha = rz / (d * q).sum(0)
            x += alpha * d
            r -= alpha * q
            z = r * J
            new = (r * z).sum(0)
            d = z + (new / rz) * d
            rz = new
        P[:, on] = x
        return P

    def density(self, X, U):
        """Density at the quadrature points, LDA, Hartree potential (from U), and H(X)."""
        dt = self.dt
        rho = torch.zeros(self.vext.shape, dtype=F64, device=DEV)
        for c in range(X.shape[1]):
            x = torch.where(dt >= 0, X[dt.clamp(min=0), c], X.new_zeros(()))
            rho += 2.0 * (x @ self.bary.T) ** 2
        eps, vxc = _lda(rho)
        w = 0.25 * self.vol[:, None]
        b = torch.zeros(self.n, dtype=F64, device=DEV)
        b.index_add_(0, dt[dt >= 0], ((w * rho) @ self.bary)[dt >= 0])
        U = self._poisson(4.0 * math.pi * b, U)
        u = torch.where(dt >= 0, U[dt.clamp(min=0)], U.new_zeros(()))
        self.H = self.Lh + self._potential(self.vext + u @ self.bary.T + vxc)
        parts = torch.stack([(w * rho).sum(), (w * eps * rho).sum(), (w * vxc * rho).sum(), 0.5 * (U @ b)])
        return rho, eps, vxc, U, parts

    def _poisson(self, rhs, U):
        col, L = self.col.clamp(min=0), 2.0 * self.Lh
        U = U.clone()
        mul = lambda x: (L * x[col]).sum(1)   # noqa: E731
        r = rhs - mul(U)
        z = r / self.lhd
        d, rz, stop = z.clone(), r @ z, 1e-28 * float(rhs @ rhs)
        for k in range(4000):
            if k % 25 == 0 and float(r @ r) <= stop:
                break
            q = mul(d)
            alpha = rz / (d @ q)
            U += alpha * d
            r -= alpha * q
            z = r / self.lhd
            new = r @ z
            d = z + (new / rz) * d
            rz = new
        return U


def _lda(rho):
    """Slater exchange and the Perdew-Wang 1992 correlation, unpolarized."""
    ok = rho > 1e-30
    r = torch.where(ok, rho, rho.new_ones(()))
    k = (3.0 * r / math.pi) ** (1.0 / 3.0)
    rs = (3.0 / (4.0 * math.pi * r)) ** (1.0 / 3.0)
    A, a1, b1, b2, b3, b4 = 0.031091, 0.21370, 7.5957, 3.5876, 1.6382, 0.49294
    s = rs.sqrt()
    den = 2 * A * (b1 * s + b2 * rs + b3 * rs * s + b4 * rs * rs)
    dden = A * (b1 / s + 2 * b2 + 3 * b3 * s + 4 * b4 * rs)
    lg = torch.log1p(1.0 / den)
    pre = -2 * A * (1 + a1 * rs)
    ec = pre * lg
    dec = -2 * A * a1 * lg - pre * dden / (den * den + den)
    zero = rho.new_zeros(())
    return torch.where(ok, -0.75 * k + ec, zero), torch.where(ok, -k + ec - rs / 3 * dec, zero)


def _pcal(m, case, X, Enuc):
    """The iterations of Algorithm PCAL with the paper preconditioner and BB2 steps, beta = 1."""
    p = case["p"]
    eye = torch.eye(p, dtype=F64, device=DEV)
    S = X.T @ m.times(m.B, X)
    Lc = torch.linalg.cholesky(0.5 * (S + S.T))
    X = X @ torch.linalg.solve_triangular(Lc, eye, upper=False).T
    U = torch.zeros(m.n, dtype=F64, device=DEV)
    Xp = Pp = kkt0 = None
    log = []
    for k in range(case["steps"] + 1):
        if case["scf"]:
            _, _, _, U, parts = m.density(X, U)
        HX, BX = m.times(m.H, X, m.B)
        S, L0 = X.T @ BX, X.T @ HX
        S, L0 = 0.5 * (S + S.T), 0.5 * (L0 + L0.T)
        kkt, fea = (HX - BX @ L0).norm(), (S - eye).norm()
        kkt0 = kkt if kkt0 is None else kkt0
        if case["scf"]:
            energy = 2.0 * L0.trace() - parts[3] - parts[2] + parts[1] + Enuc
        else:
            energy = torch.linalg.solve(S, L0).trace()
        if k == case["steps"]:
            log.append([float(v) for v in (energy, kkt, fea, (kkt + fea) / kkt0, eta)])
            break
        lam = L0 + torch.diag((L0 - S @ L0 + S @ (S - eye)).diagonal())
        P = m.solve(lam.diagonal(), HX + BX @ ((S - eye) - lam))
        if k == 0:
            eta0 = eta = P.norm() / X.norm()
        else:
            Y, D = P - Pp, X - Xp
            eta = ((Y * Y).sum() / (D * Y).sum().abs()).clamp(1e-8 * eta0, 1e8 * eta0)
        log.append([float(v) for v in (energy, kkt, fea, (kkt + fea) / kkt0, eta)])
        Xp, Pp = X, P
        X = X - P / eta
        X = X / (X * m.times(m.B, X)).sum(0).sqrt()
    return X, log


def _features(m, G):
    node = torch.stack([m.lhd.log(), m.bd.log(), (m.hd() - m.lhd) / m.bd], 1)
    rms = (G * G).mean(0).sqrt()
    return torch.cat([node[:, None, :].expand(-1, G.shape[1], -1), (G / rms)[..., None]], 2)


def _net(w, norm, F, heads):
    """tanh network of 32 units; heads outputs."""
    x = (F - norm[:4]) / norm[4:]
    h = torch.tanh(x @ w[:128].reshape(32, 4).T + w[128:160])
    return h @ w[160:160 + 32 * heads].reshape(heads, 32).T + w[160 + 32 * heads:]


def exact(case, seed):
    kind = case["kind"]
    if kind == "gram":
        X = _block(case, seed)
        HX, BX = -2.0 * X + 3.0 * _block(case, seed, 1), 0.02 * X + 0.01 * _block(case, seed, 2)
        return X.T @ BX, X.T @ HX
    m = _System(case, seed)
    if kind == "product":
        X = _block(case, seed)
        if case["precision"] == "f32":
            X = X.float().double()
        if case["op"] == "dual":
            return m.times(m.H, X, m.B)
        lam = torch.from_numpy(_shifts(case, seed)).to(DEV)
        return torch.where(lam < 0, m.shifted(lam, X), X.new_zeros(()))
    if kind == "density":
        a, b = _orbitals(case, seed), _orbitals(case, seed, 1)
        U, out = torch.zeros(m.n, dtype=F64, device=DEV), []
        for X in (a, 0.95 * a + 0.1 * b):
            rho, eps, vxc, U, parts = m.density(X, U)
            out.append(dict(rho=rho, eps=eps, vxc=vxc, U=U, parts=parts))
        return out
    if kind == "step":
        Z, R = _nuclei(case, seed)
        d = np.linalg.norm(R[:, None] - R[None], axis=2)
        i, j = np.triu_indices(len(Z), 1)
        X, log = _pcal(m, case, _orbitals(case, seed), float(np.sum(Z[i] * Z[j] / d[i, j])))
        return dict(X=X, stats=np.array(log))
    G, lam = _block(case, seed), torch.from_numpy(_shifts(case, seed)).to(DEV)
    if kind == "solve":
        return m.solve(lam, G)
    on = lam < 0
    J = torch.where(on, 1.0 / (m.lhd[:, None] - lam * m.bd[:, None]), G.new_ones(()))
    w, norm = (torch.from_numpy(a).to(DEV).double() for a in _weights(seed, 193 if kind == "learned" else 226))
    if kind == "learned":
        out = torch.empty_like(G)
        F = _features(m, G)
        for r in range(0, m.n, 1 << 14):
            out[r:r + (1 << 14)] = _net(w, norm, F[r:r + (1 << 14)], 1)[..., 0]
        return out.exp() * J * G
    w.requires_grad_(True)
    T = lambda V: torch.where(on, m.shifted(lam, V), V)   # noqa: E731
    heads = _net(w, norm, _features(m, G), 2)
    Zb = heads[..., 0].exp() * J * G
    P = Zb + heads[..., 1] * J * (G - T(Zb))
    loss = ((0.5 * (P * T(P)).sum(0) - (G * P).sum(0)) / (G * J * G).sum(0)).sum()
    loss.backward()
    return float(loss.detach()), w.grad
