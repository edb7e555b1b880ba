"""The largest request that cronos_natural_frequencies_noalloc takes: 10 doubles per mass, two per allowed
Lanczos step, a sum per workgroup and one per 256 masses, each part padded to 32 doubles, in 2^23."""
import numpy as np
import pytest

from paper_2207_09334_amd import cronos as CR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 70, 700])
def test_largest_request(n):
    x = np.stack([0.01 * np.arange(n), np.zeros(n), np.zeros(n)], 1) + 1e-3 * np.random.default_rng(n).normal(size=(n, 3))
    ends = np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32)
    rest = np.linalg.norm(x[1:] - x[:-1], axis=1)
    sim = CR.cronos_create(x, np.full(n, 0.1), ends, np.full(n - 1, 100.0), rest, pinned=np.arange(n) == 0,
                           gravity=(0.0, 0.0, 0.0), dt=1e-4)
    pad = lambda c: (max(c, 1) + 31) // 32 * 32
    block = CR.cronos_launch_config(sim)["block_masses"]
    fixed = pad(n) + 3 * pad(3 * n) + pad(-(-n // block)) + pad(-(-n // 256))
    most = ((1 << 23) - fixed) // 2 // 32 * 32
    a = CR.cronos_natural_frequencies_noalloc(sim, n_modes=1, max_iter=most, tol=1e-6)
    b = CR.cronos_natural_frequencies(sim, n_modes=1, max_iter=most, tol=1e-6)
    assert np.array_equal(a[0], b[0], equal_nan=True) and a[1] == b[1]
    with pytest.raises(CR.CronosError) as e:
        CR.cronos_natural_frequencies_noalloc(sim, n_modes=1, max_iter=most + 32, tol=1e-6)
    assert e.value.status == CR.EINVAL
    sim.close()
