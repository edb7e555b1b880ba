"""The tridiagonal eigenvalue search where the interval that holds the eigenvalues is wider than a double
can tell: a diagonal matrix's eigenvalues are its entries, each found to one ulp."""
import numpy as np
import pytest

from paper_2207_09334_amd import cronos as CR


@pytest.mark.parametrize("count", [1, 2, 3, 5])
@pytest.mark.parametrize("low", [-1.7e308, -1e308, -5e307])
def test_interval_wider_than_the_largest_double(low, count):
    a = np.array([3.0e307, low, 1.6e308, -2.0e306, 1.2e308])
    theta, _ = CR.cronos_tridiag_smallest(a, np.zeros(4), count)
    ref = np.sort(a)[:count]
    assert np.all(np.abs(theta - ref) <= 2.0 * np.spacing(np.abs(ref)))
