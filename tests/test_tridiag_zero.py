"""The lowest eigenvector of a tridiagonal matrix that is zero, or tiny: the
ground state of a sector in which H vanishes (one row of the 4-site ring at
momentum pi/2) is asked for like any other."""
import numpy as np
import pytest

from paper_1804_05028_amd import _lib as L


@pytest.mark.parametrize("m", [1, 2, 5])
@pytest.mark.parametrize("scale", [0.0, 1e-300, 1e-200, 1.0])
def test_lowest_vector_of_a_small_matrix(m, scale):
    a, b = -scale * np.arange(m, dtype=float), 0.3 * scale * np.ones(max(m - 1, 0))
    ev, v = L.ed_tridiag_eigh(a, b)
    T = np.diag(a) + np.diag(b, 1) + np.diag(b, -1)
    assert abs(np.linalg.norm(v) - 1.0) < 1e-14
    assert np.abs(T @ v - ev[0] * v).max() <= 1e-13 * max(scale * m, 1e-130)
    assert np.all(np.diff(ev) >= 0)
