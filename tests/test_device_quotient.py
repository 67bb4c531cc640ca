"""The corrected product of rmc_math.h that stands for a division along a ray
(a / b from y = 1 / b): the correctly rounded quotient, bit for bit, over
coordinate differences (0 to 1, down to 2^-60) and direction components down
to 2^-1000, with mantissas at their ends among them."""
import ctypes
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SRC = """
#include "rmc_math.h"
extern "C" void quotients(const double *a, const double *b, double *q, long n) {
  for (long i = 0; i < n; ++i) q[i] = rmc::quotient(a[i], b[i], 1.0 / b[i]);
}
"""


def test_quotient_is_the_rounded_division(tmp_path):
    src, out = tmp_path / "q.cpp", str(tmp_path / "q.so")
    src.write_text(SRC)
    p = subprocess.run([HIPCC, "-O2", "-fPIC", "-shared", "-I" + os.path.join(ROOT, "paper_2001_11252_amd", "csrc"),
                        "-o", out, str(src)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-3000:]
    lib = ctypes.CDLL(out)
    rng = np.random.default_rng(7)
    n = 400_000
    ends = np.array([1.0, 1.0 + 2.0**-52, 2.0 - 2.0**-52, 2.0 - 2.0**-51, 1.5, 1.5 - 2.0**-52, 4.0 / 3.0])

    def mantissas(m):
        x = 1.0 + rng.integers(0, 2**52, m) * 2.0**-52
        x[: m // 4] = rng.choice(ends, m // 4)
        return rng.permutation(x)

    a = mantissas(n) * np.ldexp(1.0, -rng.integers(1, 61, n))
    b = mantissas(n) * np.ldexp(1.0, -rng.integers(1, 12, n)) * rng.choice([-1.0, 1.0], n)
    b[: n // 8] = np.ldexp(b[: n // 8], -rng.integers(0, 985, n // 8))
    b[-1000:] = rng.choice([-1.0, 1.0], 1000)
    a *= rng.choice([-1.0, 1.0], n)
    a[:1000] = 0.0
    # differences of coordinates as the walk forms them: faces of levels 0 to 16 less a point
    m = n // 4
    lev = rng.integers(0, 17, m)
    a[-m:] = rng.integers(0, 2**16, m) % (2**lev + 1) * np.ldexp(1.0, -lev) - rng.random(m)
    q = np.empty(n)
    ptr = lambda x: np.ascontiguousarray(x).ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    a, b = np.ascontiguousarray(a), np.ascontiguousarray(b)
    lib.quotients(ptr(a), ptr(b), ptr(q), ctypes.c_long(n))
    assert np.abs(b).min() > 2.0**-1000
    assert np.array_equal(q, a / b)
