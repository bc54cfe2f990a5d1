"""The 1-D matrices of a uniform mesh are symmetric under reflection to the
rounding of the knots, 16 n eps of their largest entry: the split into even and
odd eigenvectors reads one half of them and refuses anything larger."""
import numpy as np
import pytest


@pytest.mark.parametrize("degree", [1, 2, 3, 4])
def test_matrices_are_symmetric_under_reflection(degree):
    import paper_1802_09277_amd as sth
    for n_elem in (2, 3, 7, 30, 54, 59, 83, 96, 127, 200, 257):
        F = sth.host_factors(level=0, dim=2, n_elem=n_elem, degree=degree, n_slabs=2, n_elem_t=1)
        n = len(F["mu"])
        for A in (F["M1"], F["K1"]):
            assert np.abs(A - A[::-1, ::-1]).max() <= 16 * n * 2.2e-16 * np.abs(A).max()
