"""The least squares of a GMRES cycle (la::lstsq) where the Krylov space ended:
the Hessenberg matrix has columns of zeros behind the last vector, on CPU."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def la():
    d = tempfile.mkdtemp()
    so = os.path.join(d, "libla.so")
    src = [os.path.join(ROOT, "tests", "native", "smallla_capi.cpp"),
           os.path.join(ROOT, "paper_1903_06986_amd", "csrc", "smallla.cpp")]
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so] + src, check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("p,t", [(10, 1), (10, 3), (9, 4), (12, 11), (4, 0)])
def test_zero_columns_get_the_coefficient_zero(la, p, t):
    rng = np.random.default_rng(p + t)
    H = np.zeros((p + 1, p), complex, order="F")
    H[:, :t] = np.triu(rng.standard_normal((p + 1, t)) + 1j * rng.standard_normal((p + 1, t)), -1)
    if t:
        H[t, t - 1] = 0  # the space is invariant
    if t + 4 < p:
        H[t + 4, t + 4] = 1  # a block that starts at a zero vector
    b = np.zeros(p + 1, complex)
    b[0] = 2.5
    x = np.zeros(p, complex)
    arg = [v.ctypes.data_as(ctypes.c_void_p) for v in (H, b, x)]
    la.la_lstsq(p + 1, p, *arg)
    assert np.all(np.isfinite(x)) and np.all(x[t:] == 0)
    if t:
        ref = np.linalg.lstsq(H[:, :t], b, rcond=None)[0]
        assert np.abs(x[:t] - ref).max() < 1e-12 * np.abs(ref).max() * np.linalg.cond(H[:t, :t])
