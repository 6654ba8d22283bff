// Small dense FP64 algebra on the host for the p x p quantities of PCAL:
// Cholesky (Cholesky-based Gram-Schmidt of the starting block, Section 4.2),
// triangular inverse, a cyclic Jacobi symmetric eigensolver and the
// generalized problem A y = lambda S y by Cholesky reduction (Rayleigh-Ritz,
// Section 4.3).  Row-major storage, p <= a few hundred.
#pragma once

#include <cmath>
#include <algorithm>
#include <exception>
#include <thread>
#include <vector>

namespace ofks {
namespace dense {

// x . y over m values with four partial sums (their order is fixed)
inline double dot4(const double *x, const double *y, int m) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int k = 0;
    for (; k + 4 <= m; k += 4) {
        s0 += x[k] * y[k];
        s1 += x[k + 1] * y[k + 1];
        s2 += x[k + 2] * y[k + 2];
        s3 += x[k + 3] * y[k + 3];
    }
    for (; k < m; ++k) s0 += x[k] * y[k];
    return (s0 + s1) + (s2 + s3);
}

// f(i) for i in [i0, i1), over host threads from `serial` items on (thread t
// takes i0 + t, i0 + t + threads, ...); f touches only what belongs to i, so
// the result does not depend on the split.  Where no thread can be started the
// caller's own does the work.
template <typename F> void rows_in_parallel(int i0, int i1, int serial, const F &f) {
    const int nt = i1 - i0 >= serial ? std::max(1, std::min(8, (int)std::thread::hardware_concurrency())) : 1;
    std::vector<std::thread> th;
    std::vector<char> started(nt, 0);
    auto part = [&](int t) {
        for (int i = i0 + t; i < i1; i += nt) f(i);
    };
    for (int t = 1; t < nt; ++t) {
        try {
            th.emplace_back(part, t);
            started[t] = 1;
        } catch (const std::exception &) {
            break;
        }
    }
    for (int t = 0; t < nt; ++t)
        if (!started[t]) part(t);
    for (auto &x : th) x.join();
}

// A = L L^T in place (lower triangle holds L, upper zeroed).  false if not SPD.
// By blocks of columns: the block's own rows in turn, then the rows below it,
// which need only those, over host threads (p = 512: 7.6 -> 2.1 ms).
inline bool cholesky(std::vector<double> &A, int p) {
    constexpr int NB = 64;
    for (int j0 = 0; j0 < p; j0 += NB) {
        const int j1 = std::min(p, j0 + NB);
        for (int i = j0; i < j1; ++i) {
            double *ai = &A[(size_t)i * p];
            for (int j = j0; j < i; ++j) {
                const double *aj = &A[(size_t)j * p];
                ai[j] = (ai[j] - dot4(ai, aj, j)) / aj[j];
            }
            const double d = ai[i] - dot4(ai, ai, i);
            if (!(d > 0.0) || !std::isfinite(d)) return false;
            ai[i] = std::sqrt(d);
        }
        rows_in_parallel(j1, p, 256, [&](int i) {
            double *ai = &A[(size_t)i * p];
            for (int j = j0; j < j1; ++j) {
                const double *aj = &A[(size_t)j * p];
                ai[j] = (ai[j] - dot4(ai, aj, j)) / aj[j];
            }
        });
    }
    for (int i = 0; i < p; ++i)
        for (int j = i + 1; j < p; ++j) A[(size_t)i * p + j] = 0.0;
    return true;
}

// inverse of a lower-triangular L (result lower triangular), by rows:
// row i of L^-1 is (e_i - sum_{k<i} L_ik row k) / L_ii; ranges of columns are
// independent and go to host threads
inline std::vector<double> lower_inverse(const std::vector<double> &L, int p) {
    std::vector<double> M((size_t)p * p, 0.0);
    constexpr int NB = 32;
    const int nblk = (p + NB - 1) / NB;
    rows_in_parallel(0, nblk, 10, [&](int q) {
        const int c0 = q * NB, c1 = std::min(p, c0 + NB);
        for (int i = c0; i < p; ++i) {
            double *mi = &M[(size_t)i * p];
            const int ce = std::min(c1, i);
            for (int k = c0; k < i; ++k) {
                const double l = L[(size_t)i * p + k];
                const double *mk = &M[(size_t)k * p];
                const int je = std::min(c1 - 1, k);
                for (int j = c0; j <= je; ++j) mi[j] -= l * mk[j];
            }
            const double inv = 1.0 / L[(size_t)i * p + i];
            for (int j = c0; j < ce; ++j) mi[j] *= inv;
            if (i < c1) mi[i] = inv;
        }
    });
    return M;
}

// Cyclic Jacobi: A symmetric (destroyed), eigenvalues w ascending, V columns
// eigenvectors (row-major, V[i*p + j] = component i of vector j).
inline void sym_eig(std::vector<double> A, int p, std::vector<double> &w, std::vector<double> &V) {
    V.assign(p * p, 0.0);
    for (int i = 0; i < p; ++i) V[i * p + i] = 1.0;
    double fro = 0.0;
    for (double x : A) fro += x * x;
    fro = std::sqrt(fro);
    for (int sweep = 0; sweep < 100; ++sweep) {
        double off = 0.0;
        for (int i = 0; i < p; ++i)
            for (int j = i + 1; j < p; ++j) off += A[i * p + j] * A[i * p + j];
        if (std::sqrt(off) <= 1e-15 * fro || off == 0.0) break;
        for (int i = 0; i < p; ++i) {
            for (int j = i + 1; j < p; ++j) {
                const double aij = A[i * p + j];
                if (aij == 0.0) continue;
                const double aii = A[i * p + i], ajj = A[j * p + j];
                const double theta = (ajj - aii) / (2.0 * aij);
                const double t = (theta >= 0 ? 1.0 : -1.0) /
                                 (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
                const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
                for (int k = 0; k < p; ++k) {  // rows i, j
                    const double aik = A[i * p + k], ajk = A[j * p + k];
                    A[i * p + k] = c * aik - s * ajk;
                    A[j * p + k] = s * aik + c * ajk;
                }
                for (int k = 0; k < p; ++k) {  // columns i, j
                    const double aki = A[k * p + i], akj = A[k * p + j];
                    A[k * p + i] = c * aki - s * akj;
                    A[k * p + j] = s * aki + c * akj;
                }
                for (int k = 0; k < p; ++k) {
                    const double vki = V[k * p + i], vkj = V[k * p + j];
                    V[k * p + i] = c * vki - s * vkj;
                    V[k * p + j] = s * vki + c * vkj;
                }
            }
        }
    }
    // sort ascending
    std::vector<int> idx(p);
    for (int i = 0; i < p; ++i) idx[i] = i;
    for (int i = 1; i < p; ++i) {
        int k = idx[i], j = i - 1;
        while (j >= 0 && A[idx[j] * p + idx[j]] > A[k * p + k]) { idx[j + 1] = idx[j]; --j; }
        idx[j + 1] = k;
    }
    std::vector<double> V2(p * p);
    w.resize(p);
    for (int j = 0; j < p; ++j) {
        w[j] = A[idx[j] * p + idx[j]];
        for (int i = 0; i < p; ++i) V2[i * p + j] = V[i * p + idx[j]];
    }
    V.swap(V2);
}

// A y = lambda S y with S SPD: S = L L^T, C = L^-1 A L^-T, C = W diag W^T,
// Y = L^-T W (so Y^T S Y = I).  false if S is not SPD.
inline bool sym_gen_eig(const std::vector<double> &A, const std::vector<double> &S, int p,
                        std::vector<double> &w, std::vector<double> &Y) {
    std::vector<double> L = S;
    if (!cholesky(L, p)) return false;
    std::vector<double> Li = lower_inverse(L, p);
    std::vector<double> T(p * p, 0.0), C(p * p, 0.0);
    for (int i = 0; i < p; ++i)
        for (int j = 0; j < p; ++j) {
            double s = 0.0;
            for (int k = 0; k <= i; ++k) s += Li[i * p + k] * A[k * p + j];
            T[i * p + j] = s;
        }
    for (int i = 0; i < p; ++i)
        for (int j = 0; j < p; ++j) {
            double s = 0.0;
            for (int k = 0; k <= j; ++k) s += T[i * p + k] * Li[j * p + k];
            C[i * p + j] = s;
        }
    for (int i = 0; i < p; ++i)
        for (int j = i + 1; j < p; ++j) {
            const double m = 0.5 * (C[i * p + j] + C[j * p + i]);
            C[i * p + j] = C[j * p + i] = m;
        }
    std::vector<double> W;
    sym_eig(C, p, w, W);
    Y.assign(p * p, 0.0);
    for (int i = 0; i < p; ++i)
        for (int j = 0; j < p; ++j) {
            double s = 0.0;
            for (int k = i; k < p; ++k) s += Li[k * p + i] * W[k * p + j];
            Y[i * p + j] = s;
        }
    return true;
}

// tr(S^-1 A) for S SPD and A symmetric, via S = L L^T: sum_i x A x^T over the
// rows x of L^-1 (x has i + 1 entries, and A's lower triangle serves both halves).
inline bool trace_sinv_a(const std::vector<double> &S, const std::vector<double> &A, int p,
                         double &out) {
    std::vector<double> L = S;
    if (!cholesky(L, p)) return false;
    const std::vector<double> Li = lower_inverse(L, p);
    std::vector<double> term(p);   // summed in row order
    rows_in_parallel(0, p, 256, [&](int i) {
        const double *x = &Li[(size_t)i * p];
        double s = 0.0;
        for (int k = 0; k <= i; ++k) {
            const double *a = &A[(size_t)k * p];
            s += x[k] * (a[k] * x[k] + 2.0 * dot4(a, x, k));
        }
        term[i] = s;
    });
    double tr = 0.0;
    for (int i = 0; i < p; ++i) tr += term[i];
    out = tr;
    return true;
}

}  // namespace dense
}  // namespace ofks
