"""The interface box grown by some cells, which bounds the reverse stencils of
the differentiation window (fslbm_adjoint.hpp, GrownBox), against its
definition: every box on one axis over the extents that the models take, the
ones that start at the first planes and cross the low periodic face among
them. Host code only, compiled from the library's header.
"""
import os
import subprocess

import pytest

from paper_1509_07691_amd import build_lib

HERE = os.path.dirname(os.path.abspath(__file__))


def test_grown_box_matches_its_definition(tmp_path):
    try:
        cc = build_lib.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    exe = str(tmp_path / "grown_box")
    subprocess.run([cc, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-result",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I",
                    build_lib.INCLUDE, "-I", build_lib.CSRC, os.path.join(HERE, "grown_box_driver.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]
    assert " 0 wrong" in r.stdout
