"""The production curved-spacetime step's sine and cosine of a midpoint, taken
from those of the step's start where that is as accurate, on the host against
extended precision.

Bound: units of 2^-53 of the value.  The evaluated pair is within 2; a turned
sine adds a correction of at most half its start (error 2 + 1) to a start of at
most twice the result (2 x 2), and is rounded (1/2): below 8.  The cosine, of
which no power is divided by, is held to 8 units of 1."""
import ctypes

import numpy as np
import pytest

from host_arith import compile_host

SOURCE = """
#define GCB_ARITH_NS arith_fast
#define GCB_FAST_ARITH 1
#include <hip/hip_runtime.h>
#include "gcb_gr.hpp"
extern "C" void near(const double* th0, const double* th1, long n, double* sn, double* cs) {
    for (long i = 0; i < n; ++i) {
        double s0, c0;
        gcb::gr::sincos_fast(th0[i], s0, c0);
        gcb::gr::sincos_near(th1[i], th1[i] - th0[i], s0, c0, sn[i], cs[i]);
    }
}
"""


@pytest.fixture(scope="module")
def near(tmp_path_factory):
    lib = compile_host(str(tmp_path_factory.mktemp("turn")), SOURCE, "-ffp-contract=fast")

    def call(th0, th1):
        out = np.empty((2, th0.size))
        p = [a.ctypes.data_as(ctypes.c_void_p) for a in (th0, th1, out[0], out[1])]
        lib.near(p[0], p[1], ctypes.c_long(th0.size), p[2], p[3])
        return out
    return call


@pytest.mark.parametrize("end", [1e-3, 1e-4, 1e-6, "anywhere"])
@pytest.mark.parametrize("pole", ["north", "south"])
def test_midpoint_sine_keeps_its_relative_accuracy(near, end, pole):
    rng = np.random.default_rng(11)
    n = 20000
    if end == "anywhere":
        th0 = rng.uniform(1e-3, np.pi - 1e-3, n)
        th1 = np.clip(th0 + rng.uniform(-0.08, 0.08, n), 1e-6, np.pi - 1e-6)
    else:
        th0 = rng.uniform(1e-3, 0.06, n)
        th1 = end * rng.uniform(0.5, 2.0, n)
        if pole == "south":
            th0, th1 = np.pi - th0, np.pi - th1
    sn, cs = near(th0, th1)
    x = th1.astype(np.longdouble)
    unit = 2.0 ** -53
    es = np.max(np.abs(sn - np.sin(x)) / np.abs(np.sin(x))) / unit
    ec = np.max(np.abs(cs - np.cos(x))) / unit
    print(f"{pole} {end}: sine {float(es):.2f}, cosine {float(ec):.2f} units")
    assert es <= 8.0 and ec <= 8.0
