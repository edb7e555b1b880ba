"""Several lanes per mass on bodies whose incidence counts cover every remainder and group of
the lane kernels (0 to 45 springs a mass, single and several rows per lane), passive and
actuated: the step's own force m v' / dt after one step from rest against the FP64 oracle.  The
bar is the force bar of the other parity tests, 1e-5 of the summed magnitudes at each mass."""
import numpy as np
import pytest

from oracle import physics as P
from paper_2207_09334_amd import cronos as CR
from tests.gpu_common import as_f32, force_scale, say

pytestmark = pytest.mark.gpu


def _body(degree, seed):
    """300 points in a 5 cm cube: every pair of the first 150 whose index distance modulo 150 is
    at most degree // 2 (about `degree` springs each), the next 60 in a chain, the rest free."""
    rng = np.random.default_rng(seed)
    x = rng.uniform(0.0, 0.05, (300, 3))
    ends = [(i, (i + d) % 150) for d in range(1, degree // 2 + 1) for i in range(150)]
    ends += [(i, i + 1) for i in range(150, 209)]
    ends = np.array([(min(e), max(e)) for e in ends], np.int32)
    return x, np.unique(ends, axis=0)


@pytest.mark.parametrize("lanes", [2, 4])
@pytest.mark.parametrize("actuated", [False, True])
@pytest.mark.parametrize("degree", [2, 6, 14, 18, 26, 32, 38, 45])
def test_one_step_forces(lanes, actuated, degree):
    say(f"case: lanes {lanes}, actuated {actuated}, degree {degree}")
    x, ends = _body(degree, degree)
    k, rest = np.full(len(ends), 50.0), np.where(np.arange(len(ends)) % 3 == 0, 0.02, 0.03)
    mass, dt = np.full(len(x), 0.1), 1e-4
    group = (np.arange(len(ends)) % 4 - 1).astype(np.int16) if actuated else None
    phase, amp = np.array([0.3, 1.1, 2.5]), np.array([0.1, 0.2, 0.05])
    sim = CR.cronos_create(x, mass, ends, k, rest, group=group, n_groups=3 if actuated else 0, dt=dt, block_masses=64,
                           lanes_per_mass=lanes)
    if actuated:
        CR.cronos_set_actuation(sim, phase, amp, 2.0)
    assert CR.cronos_launch_config(sim)["lanes_per_mass"] == lanes
    x0, _, _ = CR.cronos_read_state(sim)
    CR.cronos_step(sim, 1)
    _, v, _ = CR.cronos_read_state(sim)
    ref = as_f32(P.System(mass=mass, pinned=np.zeros(len(x), bool), ends=ends, k=k, rest=rest,
                          gidx=np.full(len(ends), -1) if group is None else group.astype(np.int64),
                          gravity=np.array([0.0, 0.0, -9.81]), damping=0.0, dt=dt, phase=phase, amp=amp, freq=2.0))
    err = np.linalg.norm(mass[:, None] * v / dt - P.forces(ref, x0, 0.0), axis=1) / force_scale(ref, x0, 0.0)
    say(f"  force error {err.max():.2e}")
    assert err.max() <= 1e-5
    sim.close()
