"""Explicit entries with four lanes per mass need six entry rows a mass on average.  Slices of every number of
rows from none on beside long ones, and bodies on either side of six rows, step bitwise as with one lane."""
import numpy as np
import pytest

from tests.test_gpu_quads import _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("actuated", [False, True])
@pytest.mark.parametrize("rows", [list(range(0, 10)) + [60, 63], [5], [6], [0, 12], [0, 11]], ids=str)
def test_few_and_many_rows(rows, actuated):
    rng = np.random.default_rng(len(rows))
    x, ends = [], []
    for s, d in enumerate(rows):   # one hub with d leaves in each slice
        x.append(rng.uniform(-0.4, 0.4, (64, 3)) + np.array([2.0 * s, 0.0, 0.0]))
        ends += [(64 * s, 64 * s + 1 + j) for j in range(d)]
    _same(np.concatenate(x), np.array(ends, np.int32).reshape(-1, 2), 0.45 + 0.1 * (np.arange(len(ends)) % 3), actuated)
