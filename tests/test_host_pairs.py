"""Conjugate partners of Ritz values (la::pair_conjugates, smallla.cpp), on
CPU: the left eigenvector of a mode in eigenvalue subtraction is made from its
partner's Ritz vector, so a real mode has to be its own."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def pair():
    d = tempfile.mkdtemp()
    so = os.path.join(d, "libpairs.so")
    src = [os.path.join(ROOT, "tests", "native", "pairs_capi.cpp"),
           os.path.join(ROOT, "paper_1903_06986_amd", "csrc", "smallla.cpp")]
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so] + src, check=True)
    lib = ctypes.CDLL(so)

    def call(w):
        w = np.array(w, dtype=np.complex128)
        p = np.zeros(len(w), dtype=np.int32)
        lib.la_pair_conjugates(len(w), w.ctypes.data_as(ctypes.c_void_p), p.ctypes.data_as(ctypes.c_void_p))
        return w, list(p)
    return call


@pytest.mark.parametrize("gap", [0.0, 2e-16, 5e-14])
@pytest.mark.parametrize("im", [0.0, 1e-17, 3e-15])
def test_equal_real_values_keep_their_own_vectors(pair, gap, im):
    """Two real values, equal or apart by less than the pairing's 1e-13, with
    imaginary parts of rounding's size: neither is the other's conjugate."""
    w = [0.7 + 0.2j, 0.5 + 1j * im, 0.9, 0.5 * (1 + gap) - 1j * im, 0.7 - 0.2j]
    got, partner = pair(w)
    assert partner == [4, 1, 2, 3, 0]
    np.testing.assert_array_equal(got[[1, 2, 3]], np.array(w)[[1, 2, 3]])


def test_converged_pairs_become_exactly_conjugate(pair):
    a, b = 0.31 + 0.02j, 0.31 + 1e-11j
    w = [a * (1 + 4e-14), 0.2, b, np.conj(a), np.conj(b) * (1 - 3e-14), 0.6 + 0.1j, (0.6 - 0.1j) * (1 + 1e-9)]
    got, partner = pair(w)
    assert partner == [3, 1, 4, 0, 2, 6, 5]  # an unconverged pair's values are partners too
    assert got[0] == np.conj(got[3]) and got[2] == np.conj(got[4])
    np.testing.assert_array_equal(got[[1, 5, 6]], np.array(w)[[1, 5, 6]])
    assert np.abs(got - w).max() < 1e-13
