"""Springs of zero length in every step form: masses that coincide pull on each other with nothing
(the force is a finite factor times a zero difference), and padding entries (a mass linked to
itself with k = 0) add nothing.  With no other force than gravity every velocity after one step is
exactly the FP32 product g dt, and a pair a small distance apart feels its spring."""
import numpy as np
import pytest

from paper_2207_09334_amd import cronos as CR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags,lanes", [(0, 1), (0, 2), (0, 4), (CR.WIDE_ENTRIES, 1), (CR.NO_TABLE, 1), (CR.SPLIT, 1),
                                         (CR.RESIDENT, 1)])
@pytest.mark.parametrize("rest", [1e-6, 0.01, 1.0])
def test_coincident_masses(flags, lanes, rest):
    n = 70   # a wavefront and six more masses; masses 2q and 2q + 1 coincide, the last two are apart
    x = np.repeat(np.linspace(0.0, 0.7, n // 2)[:, None], 2, axis=0) * np.array([[1.0, 0.5, 0.25]])
    x[-1, 0] += rest * 2.0
    ends = np.arange(n, dtype=np.int32).reshape(-1, 2)
    sim = CR.cronos_create(x, np.full(n, 0.1), ends, np.full(len(ends), 1e4), np.full(len(ends), rest), dt=1e-4,
                           flags=flags | CR.ALLOW_UNSTABLE, lanes_per_mass=lanes, block_masses=64 if lanes > 1 else 128)
    x0, _, _ = CR.cronos_read_state(sim)   # as the device holds them
    CR.cronos_step(sim, 1)
    _, v, _ = CR.cronos_read_state(sim)
    free = np.array([0.0, 0.0, np.float32(1e-4) * np.float32(-9.81)], np.float32)
    assert np.array_equal(v[:-2].astype(np.float32), np.tile(free, (n - 2, 1)))
    kick = 1e4 * (x0[-1, 0] - x0[-2, 0] - np.float32(rest)) * 1e-4 / 0.1   # k (l - rest) dt / m, inwards
    assert v[-2, 0] == pytest.approx(kick, rel=1e-2) and v[-1, 0] == pytest.approx(-kick, rel=1e-2)
    sim.close()
