"""Distances along a ray by the corrected product of rmc_math.h: wherever
quotient_holds() takes it, it equals the division bit for bit, for any start
in the cube (down to the smallest denormal from a face) and any direction a
caller may give (components from denormals to infinity and NaN); and ordinary
starts and directions are all taken."""
import ctypes
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SRC = """
#include "rmc_math.h"
extern "C" void distances(const double *face, const double *p, const double *k, double *t, int *holds, long n) {
  for (long i = 0; i < n; ++i) {
    holds[i] = rmc::quotient_holds(p + 3 * i, k + 3 * i);
    for (int d = 0; d < 3; ++d) {
      const double a = face[3 * i + d] - p[3 * i + d], b = k[3 * i + d];
      t[3 * i + d] = holds[i] ? rmc::quotient(a, b, 1.0 / b) : a / b;
    }
  }
}
"""


def test_distances_are_the_divisions_for_any_start_and_direction(tmp_path):
    src, out = tmp_path / "q.cpp", str(tmp_path / "q.so")
    src.write_text(SRC)
    p = subprocess.run([HIPCC, "-O2", "-fPIC", "-shared", "-I" + os.path.join(ROOT, "paper_2001_11252_amd", "csrc"),
                        "-o", out, str(src)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-3000:]
    lib = ctypes.CDLL(out)
    rng = np.random.default_rng(11)
    n = 400_000
    man = lambda *s: 1.0 + rng.integers(0, 2**52, s) * 2.0**-52  # noqa: E731
    face = rng.integers(0, 17, (n, 3)) / 16.0
    pos = rng.random((n, 3))
    k = rng.standard_normal((n, 3))
    k /= np.linalg.norm(k, axis=1, keepdims=True)
    plain = n // 2      # the rest: one odd coordinate or component, or several
    odd = n - plain
    c = rng.integers(0, 3, odd)
    r = np.arange(plain, n)
    face[r, c] = 0.0
    pos[r, c] = np.ldexp(man(odd), -rng.integers(1, 1075, odd))
    k[r, c] = np.ldexp(man(odd), -rng.integers(0, 12, odd)) * rng.choice([-1.0, 1.0], odd)
    s = rng.choice(r, odd // 2)
    k[s, rng.integers(0, 3, len(s))] = np.ldexp(man(len(s)), rng.integers(-1074, 1024, len(s)))
    s = rng.choice(r, odd // 16)
    k[s, rng.integers(0, 3, len(s))] = rng.choice([np.inf, -np.inf, np.nan, 0.0, -0.0, 5e-324, 1e308], len(s))
    s = rng.choice(r, odd // 16)
    pos[s, rng.integers(0, 3, len(s))] = rng.choice([0.0, 5e-324, 2.0**-50, 2.0**-51, 2.0**-1022, 1.0], len(s))
    t, holds = np.empty((n, 3)), np.empty(n, np.int32)
    ptr = lambda x: x.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    lib.distances(ptr(face), ptr(pos), ptr(k), ptr(t), ptr(holds), ctypes.c_long(n))
    assert holds[:plain].all() and 0.02 < holds[plain:].mean() < 0.5
    with np.errstate(all="ignore"):
        ref = (face - pos) / k
    walked = (k != 0.0) & ~np.isnan(ref)      # (axes without motion are left out)
    assert np.array_equal(t[walked].view(np.int64), ref[walked].view(np.int64))
