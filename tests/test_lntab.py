"""The basis form's table logarithm, built for the host from the header the
device code includes, against the C library's log: log-uniform arguments, the
edges of the table's intervals, arguments near 1, and the range Poisson ratios
take.

Bounds: r carries one rounding of 2^-53 |r| and the table two of its entry (the
reciprocal cancels: its logarithm is the entry's), the series truncates below
2^-58 (2^-56 relative beside x = 1) and the last two sums round once each: 4e-16 max(1, |ln x|) absolute, and
beside x = 1, where the entry is zero, 4e-16 relative."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2607_00488_amd", "csrc")

HARNESS = r"""
#include "lntab.h"
using std::fma;
static const nr::LnTable tab = nr::make_ln_table();
extern "C" void ln_many(const double* x, double* y, long n) {
    for (long i = 0; i < n; ++i) y[i] = nr::ln_tab(x[i], tab.e);
}
"""


@pytest.fixture(scope="module")
def ln(tmp_path_factory):
    d = tmp_path_factory.mktemp("lntab")
    (d / "h.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared",
                    "-I", CSRC, str(d / "h.cpp"), "-o", str(d / "libh.so")], check=True)
    lib = C.CDLL(str(d / "libh.so"))
    lib.ln_many.argtypes = [C.c_void_p, C.c_void_p, C.c_long]

    def f(x):
        x = np.ascontiguousarray(x, dtype=np.float64)
        y = np.empty_like(x)
        lib.ln_many(x.ctypes.data, y.ctypes.data, x.size)
        return y
    return f


def test_against_libm(ln):
    g = np.random.default_rng(20262)
    edges = np.concatenate([0.6875 + np.arange(161) / 512.0, 1.0 + np.arange(97) / 256.0])
    edges = np.concatenate([edges, np.nextafter(edges, 0), np.nextafter(edges, 2)])
    x = np.concatenate([np.exp(g.uniform(-700, 700, 400_000)),
                        1.0 + g.uniform(-5e-3, 5e-3, 200_000), g.uniform(1e-3, 1e3, 400_000),
                        edges, 2.0 * edges, 0.25 * edges,
                        [2.2250738585072014e-308, 1.7976931348623157e308]])
    y, ref = ln(x), np.log(x)
    err = np.abs(y - ref) / np.maximum(1.0, np.abs(ref))
    assert err.max() <= 4e-16, (err.max(), x[np.argmax(err)])
    near = np.abs(x - 1.0) < 2.0 ** -9
    rel = np.abs(y[near] - ref[near]) / np.maximum(np.abs(ref[near]), 1e-300)
    assert rel.max() <= 4e-16
    assert ln(np.array([1.0]))[0] == 0.0
