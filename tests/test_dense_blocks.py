"""The blocked, threaded p x p algebra (csrc/dense.hpp), compiled with g++, at
the edges of its blocks and thread thresholds: the Cholesky factor, the
inverse of a triangle and tr(S^-1 A) against sums in long double."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2007_14228_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "dense.hpp"
using namespace ofks;
int main(int argc, char **argv) {
    for (int q = 1; q < argc; ++q) {
        const int p = std::atoi(argv[q]);
        std::vector<double> S((size_t)p * p), A((size_t)p * p);
        unsigned long long z = 88172645463325252ull;
        auto rnd = [&]() { z ^= z << 13; z ^= z >> 7; z ^= z << 17; return (double)(z >> 11) / 9007199254740992.0 - 0.5; };
        for (int i = 0; i < p; ++i)
            for (int j = 0; j <= i; ++j) {
                S[(size_t)i * p + j] = S[(size_t)j * p + i] = i == j ? 2.0 : rnd() / p;   // 1.5 <= eigenvalues <= 2.5
                A[(size_t)i * p + j] = A[(size_t)j * p + i] = rnd();
            }
        std::vector<double> L = S;
        double tr = 0.0;
        if (!dense::cholesky(L, p) || !dense::trace_sinv_a(S, A, p, tr)) { std::printf("%d refused\n", p); return 1; }
        const std::vector<double> M = dense::lower_inverse(L, p);
        double e0 = 0.0, e1 = 0.0;
        long double ref = 0.0L, mag = 0.0L;
        for (int i = 0; i < p; ++i)
            for (int j = 0; j < p; ++j) {
                long double s = 0.0L, t = 0.0L, g = 0.0L;
                for (int k = 0; k < p; ++k) {
                    s += (long double)L[(size_t)i * p + k] * L[(size_t)j * p + k];
                    t += (long double)L[(size_t)i * p + k] * M[(size_t)k * p + j];
                    g += (long double)M[(size_t)k * p + i] * M[(size_t)k * p + j];   // (S^-1)_ij
                }
                e0 = std::max(e0, (double)std::fabs(s - S[(size_t)i * p + j]));
                e1 = std::max(e1, (double)std::fabs(t - (i == j)));
                ref += g * A[(size_t)j * p + i];
                mag += std::fabs(g * A[(size_t)j * p + i]);
            }
        S[(size_t)p * p - 1] = -1.0;
        std::printf("%d %.3e %.3e %.3e %d\n", p, e0, e1, (double)(std::fabs(tr - ref) / mag), (int)dense::cholesky(S, p));
    }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_factor_inverse_and_trace_at_block_edges(tmp_path):
    (tmp_path / "d.cpp").write_text(DRIVER)
    exe = tmp_path / "d"
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I", CSRC, str(tmp_path / "d.cpp"), "-o", str(exe)],
                   check=True)
    sizes = [1, 2, 31, 33, 63, 64, 65, 128, 255, 256, 257, 289, 320, 321]
    out = subprocess.run([str(exe)] + [str(p) for p in sizes], capture_output=True, text=True, check=True).stdout
    rows = [line.split() for line in out.splitlines()]
    assert [int(r[0]) for r in rows] == sizes
    for p, factor, inverse, trace, spd in rows:
        # dots of at most p terms of size <= 2.5, eigenvalues between 1.5 and 2.5: (p + 8) eps times a few units
        bound = 10 * (int(p) + 8) * 2.0 ** -53
        assert float(factor) <= bound and float(inverse) <= bound and float(trace) <= 4 * bound, (p, factor, inverse, trace)
        assert spd == "0"                                 # a negative last diagonal is refused
