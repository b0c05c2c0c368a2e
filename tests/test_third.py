"""The kernels' division by three (common.hpp) against the division, bit for bit,
compiled for the host: random significands over every exponent, subnormal numbers
and their edge, multiples of three and their neighbours, zeros, infinities, NaN."""
import ctypes as C
import os
import subprocess

import numpy as np

from paper_1505_04694_amd import build

SOURCE = """
#include "common.hpp"
extern "C" void thirds(const double* x, double* y, long n) {
  for (long i = 0; i < n; ++i) y[i] = pm::third(x[i]);
}
"""


def test_third_is_the_division(tmp_path):
    src, so = tmp_path / "third.hip", tmp_path / "third.so"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O2",
                    "-ffp-contract=off", "-I", build.CSRC, "-fPIC", "-shared", str(src), "-o", str(so)],
                   check=True, capture_output=True, text=True)
    rng = np.random.default_rng(1)
    bits = [rng.integers(0, 2 ** 64, 1_000_000, dtype=np.uint64),  # every exponent, both signs
            rng.integers(0, 2 ** 56, 300_000, dtype=np.uint64),    # the smallest exponents, subnormals
            rng.integers(0, 2 ** 20, 100_000, dtype=np.uint64),    # the smallest subnormals
            np.arange(0, 4096, dtype=np.uint64),
            np.uint64(0x7FF0000000000000) - np.arange(0, 4096, dtype=np.uint64)]  # infinity and the largest
    x = np.concatenate([b.view(np.float64) for b in bits])
    q = rng.uniform(1, 2, 300_000) * 2.0 ** rng.integers(-1070, 1020, 300_000)
    with np.errstate(all="ignore"):
        x = np.concatenate([x, -x, 3 * q, np.nextafter(3 * q, 0), np.nextafter(3 * q, np.inf), [0.0, -0.0, np.inf, -np.inf]])
        want = x / 3.0
    got = np.empty_like(x)
    f = C.CDLL(os.fspath(so)).thirds
    f.argtypes = [C.c_void_p, C.c_void_p, C.c_long]
    f(x.ctypes.data, got.ctypes.data, x.size)
    nan = np.isnan(x)
    assert np.array_equal(np.isnan(got), nan)
    bad = np.flatnonzero((got.view(np.uint64) != want.view(np.uint64)) & ~nan)
    assert bad.size == 0, [(x[i].hex(), got[i].hex(), want[i].hex()) for i in bad[:5]]
