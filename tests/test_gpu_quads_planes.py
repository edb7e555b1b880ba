"""Explicit entries with four lanes per mass where the choice of coordinate difference matters: a slice of
64 masses, some beside a coordinate plane and the others far from all, tied by springs stretched over
many rest lengths, whose plain difference of coordinates rounds.  One lane per mass decides for the
64 masses together; the four-lane form steps bitwise the same, whichever of the slice's masses are near."""
import numpy as np
import pytest

from paper_2207_09334_amd import cronos as CR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("actuated", [False, True])
@pytest.mark.parametrize("near", [0, 1, 5, 16, 48, 63], ids=lambda q: f"near{q}")
@pytest.mark.parametrize("axes", [(0, 1, 2), (2,)], ids=["all", "z"])
@pytest.mark.parametrize("n", [64, 100, 640])
def test_bitwise_one_lane(n, axes, near, actuated):
    rng = np.random.default_rng(n + near)
    x = rng.uniform(5.0, 60.0, (n, 3))
    beside = np.arange(n) % 64 < near
    for c in axes:
        x[beside, c] = rng.uniform(-0.5, 0.5, beside.sum())
    ends = np.array([(i, i + d) for d in (1, 5, 16) for i in range(n - d)], np.int32)
    kw = dict(dt=1e-4, damping=1e-3, block_masses=64, flags=CR.ALLOW_UNSTABLE | CR.NO_TABLE | CR.NO_SHIFT)
    if actuated:
        kw.update(group=(np.arange(len(ends)) % 5 - 1).astype(np.int16), n_groups=4)
    out = []
    for persistent in (0, 1):   # persistent workgroups take one lane per mass, on the same 64-mass slices
        sim = CR.cronos_create(x, np.full(n, 0.1), ends, np.full(len(ends), 50.0), np.full(len(ends), 0.5),
                               persistent=persistent, **kw)
        if actuated:
            CR.cronos_set_actuation(sim, [0.1, 0.7, 1.9, 3.0], [0.2, 0.1, 0.0, 0.3], 2.0)
        assert CR.cronos_launch_config(sim)["step_form"] == "explicit"
        CR.cronos_step(sim, 3)
        out.append(CR.cronos_read_state(sim)[:2])
        sim.close()
    assert np.isfinite(out[0][0]).all() and np.abs(out[0][0] - x).max() > 0
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
