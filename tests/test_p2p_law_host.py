"""The FP64 P2P force law, compiled alone for the host: how many coefficients it takes, and the weight of a pair
against 80-bit arithmetic."""
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

static double weight(const hfmm::P2PConst64 &k, double r2, double y)
{
    switch (k.ncoef) {
    case 1: return hfmm::law64_weight<1>(k, r2, 1.0, y);
    case 19: return hfmm::law64_weight<19>(k, r2, 1.0, y);
    case 22: return hfmm::law64_weight<22>(k, r2, 1.0, y);
    default: return hfmm::law64_weight<0>(k, r2, 1.0, y);
    }
}

// Largest error over its bound, and largest relative error, of n pairs at r between lo and hi (in r_cut), estimates
// of 1/r off by up to 2^-23.  Bound, in units of 2^-53: S - S_0 good to six roundings (r_cut^2 - r^2, the rounded and
// summed terms, the product), the difference from S_0 to one, f_(1) itself to four, one of them the series' end.
extern "C" void errors(double r_s, double r_cut, int split, double lo, double hi, int n, double *out)
{
    hfmm::P2PConst64 k;
    hfmm::law64_setup(r_s, r_cut, split, k);
    out[0] = out[1] = 0;
    const long double rs = (long double)r_s * k.scale, rc = (long double)r_cut * k.scale;
    for (int i = 0; i < n; ++i) {
        const double r = (double)rc * (lo + (hi - lo) * (i + 0.5) / n), r2 = r * r;
        if (!(r2 < k.rc2)) continue;
        const long double R = sqrtl((long double)r2), x = R / rc, u = R / (2 * rs);
        const long double h = split ? (1 - x) * (1 - x) * (1 + 2 * x + 3 * x * x + 1.5L * x * x * x)
                                    : erfcl(u) + 2 / sqrtl(3.14159265358979323846L) * u * expl(-u * u);
        const long double w = -h / (R * R * R), y = 1 / R;
        const double got = weight(k, r2, (double)(y * (1 + (i % 17 - 8) / 8.0L * 0x1p-23L)));
        const long double e = fabsl(got - w), newton = 1 / (R * R * R);
        const long double bound = 0x1p-53L * (6 * (newton + w - k.s0) + (newton - k.s0) + 4 * fabsl(w));
        if (e / bound > out[0]) out[0] = (double)(e / bound);
        if (e / fabsl(w) > out[1]) out[1] = (double)(e / fabsl(w));
    }
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
    d_, i_ = ctypes.c_double, ctypes.c_int
    lib.ncoef.argtypes = [d_, d_, i_]
    lib.errors.argtypes = [d_, d_, i_, d_, d_, i_, ctypes.POINTER(d_)]
    return lib


@pytest.mark.parametrize("ratio", [1.0, 2.5, 3.0, 4.0, 4.2, 4.4, 4.5, 4.6, 4.7, 4.75, 4.8, 4.9, 5.0])
def test_the_choice_depends_on_the_ratio_alone(law, ratio):
    """r_s over six decades; r_cut from r_s, and r_s from r_cut: the ratio's last bits vary."""
    rs = np.geomspace(1e-5, 10.0, 401) * (1 + 1e-3 * np.arange(401) / 401)
    got = {law.ncoef(a, a * ratio, 0) for a in rs} | {law.ncoef(a / ratio, a, 0) for a in rs}
    assert len(got) == 1 and got != {0}, got


def test_no_fit_far_beyond_five(law):
    assert {law.ncoef(a, a * r, 0) for a in (1e-4, 0.02, 0.3) for r in (5.2, 6.0, 9.0)} == {0}


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("ratio", [1.0, 3.0, 4.2, 4.5, 4.55, 4.6, 4.8, 5.0, 5.05])
@pytest.mark.parametrize("r_cut", [0.31, 1e-6, 3e-30, 0.09])
def test_a_pairs_weight_is_good_at_any_separation(law, ratio, split, r_cut):
    out = (ctypes.c_double * 2)()
    for lo, hi in [(1e-9, 1e-6), (1e-6, 0.1)] + [(k / 20, (k + 1) / 20) for k in range(2, 20)] + [(0.99, 1.0)]:
        law.errors(r_cut / ratio, r_cut, split, lo, hi, 3000, out)
        assert out[0] <= 1.0, (lo, hi, out[0], out[1])
        if split == 0:  # no more than erfc and exp are off by near the cutoff
            assert out[1] <= 3e-15, (lo, hi, out[1])


def test_alternating_force_laws_cost_little_host_time(law):
    """Two trees of different r_s, evaluated in turn: microseconds a setup (the bar is 40), not a fit's 0.2 to 0.5 ms."""
    import time
    best = 1.0
    for _ in range(5):
        t0 = time.perf_counter()
        for k in range(200):
            law.ncoef(0.02 + 1e-9 * (k & 1), 0.09 + 4.5e-9 * (k & 1), 0)
        best = min(best, (time.perf_counter() - t0) / 200)
    assert best < 40e-6, best
