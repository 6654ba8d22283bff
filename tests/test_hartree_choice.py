"""Which Hartree CG serves a plan (halo_cg_pays in csrc/halo_plan.hpp, compiled
with g++), on both sides of each of its lines."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2007_14228_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_lines(tmp_path):
    cases = [(2_000_000, 8_000_000, 1), (2_000_000, 8_000_001, 0),      # near rows have near numbers
             (70_000, 1_000_000, 1), (70_000, 1_000_001, 0),            # scattered, short and long
             (250_000, 2_000_000, 1), (249_999, 2_000_000, 0),          # between the two
             (260_000, 2_000_001, 0), (1, 1, 1)]
    calls = "".join(f"if (ofks::halo_cg_pays({n}, {h}) != {w}) return {i + 1};\n" for i, (n, h, w) in enumerate(cases))
    (tmp_path / "d.cpp").write_text('#include "halo_plan.hpp"\nint main() {\n' + calls + "return 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(tmp_path / "d.cpp"), "-o", str(tmp_path / "d")], check=True)
    assert subprocess.run([str(tmp_path / "d")]).returncode == 0
