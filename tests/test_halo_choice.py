"""Which product kernel serves a plan (csrc/halo_plan.hpp, compiled with g++): a
15-point pattern numbered along the Z-order curve, lexicographically and at
random, at the widths on both sides of each line."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as wl

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2007_14228_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include "halo_plan.hpp"
using namespace ofks;
int main(int argc, char **argv) {   // file, then p
    std::ifstream f(argv[1], std::ios::binary);
    int64_t n = 0, where = 0;
    f.read((char *)&n, 8);
    std::vector<int64_t> rp(n + 1);
    f.read((char *)rp.data(), 8 * (n + 1));
    std::vector<int32_t> col(rp[n]);
    f.read((char *)col.data(), 4 * rp[n]);
    HaloPlan P;
    if (halo_plan_build(n, rp.data(), col.data(), 192, 64, 64, P, &where) != HALO_OK) return 1;
    for (int k = 2; k < argc; ++k) {
        const int p = std::atoi(argv[k]);
        std::printf("%d %d\n", halo_product_pays(n, (int64_t)P.halo.size(), p, 8), halo_product_pays(n, (int64_t)P.halo.size(), p, 4));
    }
}
"""

WIDTHS = (1, 3, 4, 11, 23, 24, 32, 33, 63, 64, 96, 128, 129, 160, 512)


def _pattern(order):
    ax = wl.uniform_axis(-1.0, 1.0, 36)
    m = wl.kuhn_mesh(ax, ax, ax, order="lex" if order == "lex" else "morton")
    tets = m.tets
    if order == "random":
        perm = np.random.default_rng(1).permutation(len(m.xyz))
        tets = perm[tets]
        free = np.flatnonzero(m.dirichlet == 0)
        inner = np.sort(perm[free])
    else:
        inner = np.flatnonzero(m.dirichlet == 0)
    dof = np.full(len(m.xyz), -1)
    dof[inner] = np.arange(len(inner))
    t = dof[tets]
    pairs = np.concatenate([t[:, [a, b]] for a in range(4) for b in range(4)])
    pairs = np.unique(pairs[(pairs >= 0).all(1)], axis=0)
    rp = np.concatenate([[0], np.cumsum(np.bincount(pairs[:, 0], minlength=len(inner)))])
    return rp.astype(np.int64), pairs[:, 1].astype(np.int32)


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_scattered_numberings_keep_narrow_blocks_on_the_gather(tmp_path):
    (tmp_path / "d.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(tmp_path / "d.cpp"), "-o", str(tmp_path / "d")], check=True)
    got = {}
    for order in ("morton", "lex", "random"):
        rp, col = _pattern(order)
        (tmp_path / "m").write_bytes(np.int64(len(rp) - 1).tobytes() + rp.tobytes() + col.tobytes())
        out = subprocess.run([str(tmp_path / "d"), str(tmp_path / "m")] + [str(p) for p in WIDTHS], check=True,
                             capture_output=True, text=True).stdout
        rows = [tuple(int(v) for v in l.split()) for l in out.splitlines()]
        got[order] = ([p for p, r in zip(WIDTHS, rows) if r[0]], [p for p, r in zip(WIDTHS, rows) if r[1]])
    assert got["morton"] == ([p for p in WIDTHS if p >= 4], [p for p in WIDTHS if p >= 33])
    assert got["lex"] == ([p for p in WIDTHS if p >= 24], [33, 63, 129, 160, 512])
    assert got["random"] == ([64, 96, 128, 129, 160, 512], [])
