"""Host side of the FP64 P2P force law, compiled alone: how many coefficients it takes."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2006_14952_amd", "csrc")

SRC = """
#include "p2p_law.h"
extern "C" int ncoef(double r_s, double r_cut, int split)
{
    hfmm::P2PConst64 k;
    hfmm::law64_setup(r_s, r_cut, split, k);
    return k.ncoef;
}
"""

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


@pytest.fixture(scope="module")
def law(tmp_path_factory):
    d = tmp_path_factory.mktemp("law")
    (d / "law.cpp").write_text(SRC)
    so = str(d / "law.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, str(d / "law.cpp"),
                    "-o", so], check=True, capture_output=True)
    lib = ctypes.CDLL(so)
    lib.ncoef.argtypes = [ctypes.c_double, ctypes.c_double, ctypes.c_int]
    return lib


@pytest.mark.parametrize("ratio", [1.0, 2.5, 3.0, 4.0, 4.2, 4.4, 4.5, 4.6, 4.7, 4.75, 4.8, 4.9, 5.0])
def test_the_choice_depends_on_the_ratio_alone(law, ratio):
    """r_s over six decades; r_cut from r_s, and r_s from r_cut: the ratio's last bits vary."""
    rs = np.geomspace(1e-5, 10.0, 401) * (1 + 1e-3 * np.arange(401) / 401)
    got = {law.ncoef(a, a * ratio, 0) for a in rs} | {law.ncoef(a / ratio, a, 0) for a in rs}
    assert len(got) == 1 and got != {0}, got


def test_no_fit_far_beyond_five(law):
    assert {law.ncoef(a, a * r, 0) for a in (1e-4, 0.02, 0.3) for r in (5.2, 6.0, 9.0)} == {0}
