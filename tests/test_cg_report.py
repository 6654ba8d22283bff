"""The Hartree CG's report to the host (csrc/cg_report.hpp), compiled with g++:
whichever of two checks' words the host finds, a residual that stopped being
finite on the way is a divergence and one that never was is none."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2007_14228_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <limits>
#include "cg_report.hpp"
using namespace ofks;
int main() {
    const double nan = std::numeric_limits<double>::quiet_NaN(), inf = std::numeric_limits<double>::infinity();
    const double values[] = {0.0, 1e-30, 1.0, 1e300, inf, nan, -nan}, tol2 = 1e-20;
    int bad = 0;
    for (double a : values)
        for (int first = 0; first < 2; ++first) {
            const CgSeen s = cg_report_seen(cg_report_word(a, first), tol2);
            const bool finite = std::isfinite(a);
            bad += s.diverged != (!finite && !first);
            bad += s.stop != (!(a > tol2) || (!finite && !first));
            bad += finite && s.rr != a;
        }
    // two checks in turn: the host reads after the first one, perhaps the second one's word
    const double w[2] = {cg_report_word(1.0, true), cg_report_word(nan, false)};
    const CgSeen e = cg_report_seen(w[0], tol2), l = cg_report_seen(w[1], tol2);
    bad += e.stop || e.diverged || !l.stop || !l.diverged;
    static_assert(sizeof(w[0]) == 8, "one word");
    std::printf("%d\n", bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_word_tells_divergence_from_a_bad_start(tmp_path):
    (tmp_path / "d.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(tmp_path / "d.cpp"), "-o", str(tmp_path / "d")], check=True)
    assert subprocess.run([str(tmp_path / "d")], capture_output=True, text=True).returncode == 0
