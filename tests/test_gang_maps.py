"""The gang CG's cut of a lattice on the host (csrc/hub_gang.h), without a GPU.

tests/gang_maps.cpp walks every workgroup of a cut as the kernel does and compares
M M^dagger r with the plain stencil: for cuts in each direction alone and together, on
lattices down to one cell or one slice, and for the cuts that the rule picks.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_gang_maps(tmp_path):
    exe = str(tmp_path / "gang_maps")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "paper_1804_07195_amd", "csrc"),
                    os.path.join(ROOT, "tests", "gang_maps.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
