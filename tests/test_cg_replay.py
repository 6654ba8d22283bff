"""The inner CG's step (csrc/cg_step.hpp), replayed with g++ on the matrices of
small meshes: as accurate as the textbook two-term recurrence in the same type
(both against 80-bit sums), and harmless past the solution."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as wl
from oracle import fem

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2007_14228_amd", "csrc")

DRIVER = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <vector>
#include "cg_step.hpp"
using namespace ofks;
typedef long double W;
struct Csr { int64_t n, nnz; std::vector<int64_t> rp; std::vector<int32_t> col; std::vector<double> L, B; };
template <typename T> using Vec = std::vector<T>;
template <typename T> Vec<T> apply(const Csr &A, T lam, const Vec<T> &x) {
    Vec<T> y(A.n);
    for (int64_t r = 0; r < A.n; ++r) {
        T a = 0, b = 0;
        for (int64_t e = A.rp[r]; e < A.rp[r + 1]; ++e) {
            a = std::fma((T)A.L[e], x[A.col[e]], a);
            b = std::fma((T)A.B[e], x[A.col[e]], b);
        }
        y[r] = std::fma(-lam, b, a);
    }
    return y;
}
template <typename T> double dot(const Vec<T> &a, const Vec<T> &b) {
    W s = 0;
    for (size_t i = 0; i < a.size(); ++i) s += (W)a[i] * b[i];
    return (double)s;
}
template <typename T> Vec<T> two_term(const Csr &A, const Vec<T> &D, T lam, const Vec<T> &g, int m) {
    const int64_t n = A.n;
    Vec<T> x(n, 0), r = g, z(n), d(n);
    for (int64_t i = 0; i < n; ++i) d[i] = z[i] = r[i] * (T(1) / D[i]);
    W rz = 0;
    auto wdot = [&](const Vec<T> &a, const Vec<T> &b) { W s = 0; for (int64_t i = 0; i < n; ++i) s += (W)a[i] * b[i]; return s; };
    rz = wdot(r, z);
    for (int j = 0; j < m; ++j) {
        const Vec<T> q = apply<T>(A, lam, d);
        const W dq = wdot(d, q);
        const T a = dq > 0 ? (T)(rz / dq) : T(0);
        for (int64_t i = 0; i < n; ++i) {
            x[i] = std::fma(a, d[i], x[i]);
            r[i] = std::fma(-a, q[i], r[i]);
            z[i] = r[i] / D[i];
        }
        const W nx = wdot(r, z);
        const T b = rz > 0 ? (T)(nx / rz) : T(0);
        for (int64_t i = 0; i < n; ++i) d[i] = std::fma(b, d[i], z[i]);
        rz = nx;
    }
    return x;
}
template <typename T> Vec<T> replay(const Csr &A, const Vec<T> &D, T lam, const Vec<T> &g, int m) {
    const int64_t n = A.n;
    Vec<T> x(n, 0), blk[2] = {Vec<T>(n), g};   // d_j alternates; the second block starts with g
    for (int64_t i = 0; i < n; ++i) blk[0][i] = g[i] * (T(1) / D[i]);
    double rz = dot(g, blk[0]), rz0 = rz;
    T am = 0, bm = 0;
    for (int j = 0; j < m; ++j) {
        Vec<T> &d = blk[j & 1], &dm = blk[(j & 1) ^ 1];
        const Vec<T> q = apply<T>(A, lam, d);
        Vec<T> w(n);
        for (int64_t i = 0; i < n; ++i) w[i] = q[i] / D[i];
        CgCoef<T> c = cg_coef<T>(dot(d, q), dot(q, w), rz, j ? rz0 : 0.0);
        if (j + 1 == m) {
            for (int64_t i = 0; i < n; ++i) x[i] = j & 1 ? cg_x2(x[i], am, dm[i], c.alpha, d[i]) : std::fma(c.alpha, d[i], x[i]);
            break;
        }
        W s = 0;
        for (int64_t i = 0; i < n; ++i) {
            T dn;
            const double z = j ? cg_element<false>(q[i], d[i], dm[i], D[i], c.alpha, c.beta, bm, dn)
                               : cg_element<true>(q[i], d[i], dm[i], D[i], c.alpha, c.beta, bm, dn);
            s += (W)(z * z * (double)D[i]);
            if (j & 1) x[i] = cg_x2(x[i], am, dm[i], c.alpha, d[i]);
            dm[i] = dn;
        }
        if (c.old > 0.0) {
            c.beta = (T)((double)s / c.old);
            for (int64_t i = 0; i < n; ++i) dm[i] = std::fma(c.beta, d[i], dm[i]);
        }
        rz = (double)s;
        am = c.alpha;
        bm = c.beta;
    }
    return x;
}
template <typename T> void run(const Csr &A0, double lam0, int m, unsigned seed) {
    Csr A = A0;
    for (auto &v : A.L) v = (T)v;
    for (auto &v : A.B) v = (T)v;
    const T lam = (T)lam0;
    Vec<T> D(A.n), g(A.n);
    Csr X = A;
    unsigned long long z = 88172645463325252ull + seed;
    Vec<W> gw(A.n), Dw(A.n);
    for (int64_t r = 0; r < A.n; ++r) {
        for (int64_t e = A.rp[r]; e < A.rp[r + 1]; ++e)
            if (A.col[e] == r) D[r] = (T)A.L[e] - lam * (T)A.B[e], Dw[r] = (W)A.L[e] - (W)lam * A.B[e];
        double s = 0;
        for (int k = 0; k < 12; ++k) { z ^= z << 13; z ^= z >> 7; z ^= z << 17; s += (double)(z >> 11) / 9007199254740992.0; }
        g[r] = (T)(s - 6.0);
        gw[r] = g[r];
    }
    const Vec<W> ref = two_term<W>(A, Dw, (W)lam, gw, m);
    W nr = 0, e2 = 0, e3 = 0;
    const Vec<T> a = two_term<T>(A, D, lam, g, m), b = replay<T>(A, D, lam, g, m);
    for (int64_t i = 0; i < A.n; ++i) { nr += ref[i] * ref[i]; e2 += (a[i] - ref[i]) * (a[i] - ref[i]); e3 += (b[i] - ref[i]) * (b[i] - ref[i]); }
    std::printf("%d %.6e %.6e\n", (int)sizeof(T), (double)std::sqrt(e2 / nr), (double)std::sqrt(e3 / nr));
}
int main(int argc, char **argv) {   // file, m, then shifts
    std::ifstream f(argv[1], std::ios::binary);
    Csr A;
    f.read((char *)&A.n, 8);
    f.read((char *)&A.nnz, 8);
    A.rp.resize(A.n + 1); A.col.resize(A.nnz); A.L.resize(A.nnz); A.B.resize(A.nnz);
    f.read((char *)A.rp.data(), 8 * (A.n + 1)); f.read((char *)A.col.data(), 4 * A.nnz);
    f.read((char *)A.L.data(), 8 * A.nnz); f.read((char *)A.B.data(), 8 * A.nnz);
    for (int k = 3; k < argc; ++k)
        for (unsigned s = 0; s < 4; ++s) { run<double>(A, std::atof(argv[k]), std::atoi(argv[2]), 77 * s); run<float>(A, std::atof(argv[k]), std::atoi(argv[2]), 77 * s); }
}
"""

needs_gxx = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    d = tmp_path_factory.mktemp("cg")
    (d / "d.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-march=native", "-ffp-contract=off", "-std=c++17", "-Wno-unknown-pragmas", "-I", CSRC,
                    str(d / "d.cpp"), "-o", str(d / "d")], check=True)

    def go(rp, col, L, B, m, shifts):
        with open(d / "m.bin", "wb") as f:
            f.write(np.array([len(rp) - 1, len(col)], dtype=np.int64).tobytes() + rp.astype(np.int64).tobytes() +
                    col.astype(np.int32).tobytes() + L.tobytes() + B.tobytes())
        out = subprocess.run([str(d / "d"), str(d / "m.bin"), str(m)] + [str(v) for v in shifts], check=True,
                             capture_output=True, text=True).stdout
        rows = np.array([[float(v) for v in l.split()] for l in out.splitlines()])
        return {w: rows[rows[:, 0] == w][:, 1:] for w in (8, 4)}
    return go


@needs_gxx
def test_ten_steps_are_as_accurate_as_the_two_term_form(replay):
    got = {8: [], 4: []}
    for cells, grade in ((12, 2.0), (14, 4.0), (13, 5.0)):
        t = np.linspace(-1.0, 1.0, cells + 1)
        ax = 10.0 * np.sinh(grade * t) / np.sinh(grade)
        d = fem.discretize(wl.kuhn_mesh(ax, ax, ax), np.array([6.0]), np.array([[0.3, 0.1, 0.2]]))
        r = replay(d.row_ptr, d.col, 0.5 * d.L, d.B, 10, (-0.05, -0.5, -5.0, -50.0))
        for w in got:
            got[w].append(r[w][:, 1] / r[w][:, 0])
    for w, v in got.items():
        # 48 ratios that scatter by 0.12: their mean is known to 0.02
        assert np.concatenate(v).mean() <= 1.0, (w, np.concatenate(v))


@needs_gxx
@pytest.mark.parametrize("m", [1, 2, 3, 10, 40, 300])
def test_early_solutions(replay, m):
    """One, two and a few rows, independent rows and pairs, and nearly
    independent rows: the steps end the solve after one, two or a few, at once
    (then alpha d adds nothing) or by many digits a step."""
    rng = np.random.default_rng(5)
    systems = []
    for n in (1, 2, 3, 5):
        for _ in range(4):
            Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
            systems.append((Q * rng.uniform(1, 4, n)) @ Q.T)
    systems.append(np.diag(rng.uniform(1, 5, 50)))
    systems.append(np.kron(np.diag(rng.uniform(1, 3, 30)), np.array([[2.0, 0.9], [0.9, 1.5]])))
    for eps in (1e-3, 1e-5, 1e-7):
        E = rng.standard_normal((40, 40))
        systems.append(np.diag(rng.uniform(1, 5, 40)) + eps * (E + E.T))
    for A in systems:
        n = len(A)
        rp, col = np.arange(0, n * n + 1, n), np.tile(np.arange(n), n)
        r = replay(rp, col, ((A + A.T) / 2).ravel(), np.zeros(n * n), m, (-1.0,))
        for w, eps in ((8, 2.0 ** -53), (4, 2.0 ** -24)):
            if m > 1 and n < m and m > 3:   # past the solution the 80-bit recurrence only polishes it
                assert np.all(r[w][:, 1] <= 8 * r[w][:, 0] + 16 * eps), (n, w, r[w])
            else:                            # a few times the recurrence's own error
                assert np.all(r[w][:, 1] <= 4 * r[w][:, 0] + 8 * eps), (n, w, r[w])
