"""Explicit entries with four lanes per mass (64-mass workgroups of small bodies) against one lane (256-mass
workgroups, and the persistent form): bitwise the same steps, for every remainder of rows per quad, past
the rows that are loaded up front, passive and actuated, and at the size where the choice changes."""
import numpy as np
import pytest

from paper_2207_09334_amd import cronos as CR

pytestmark = pytest.mark.gpu


def _same(x, ends, rest, actuated, near_plane=False):
    out = []
    for kw in (dict(block_masses=64), dict(block_masses=256), dict(block_masses=64, persistent=1)):
        if actuated and len(ends):
            kw.update(group=(np.arange(len(ends)) % 5 - 1).astype(np.int16), n_groups=4)
        sim = CR.cronos_create(x, np.full(len(x), 0.1), ends, np.full(len(ends), 500.0), rest, dt=1e-4, damping=1e-3,
                               ground=True, ground_k=1e4, ground_mu=0.5, flags=CR.ALLOW_UNSTABLE | CR.NO_TABLE, **kw)
        if actuated and len(ends):
            CR.cronos_set_actuation(sim, [0.1, 0.7, 1.9, 3.0], [0.2, 0.1, 0.0, 0.3], 2.0)
        assert CR.cronos_launch_config(sim)["step_form"] == "explicit"
        CR.cronos_step(sim, 5)
        out.append(CR.cronos_read_state(sim)[:2])
        sim.close()
    for o in out[1:]:
        assert np.array_equal(out[0][0], o[0]) and np.array_equal(out[0][1], o[1])
    assert np.isfinite(out[0][0]).all()


@pytest.mark.parametrize("actuated", [False, True])
@pytest.mark.parametrize("rows", [list(range(0, 10)), [27, 28, 29, 30], [63], [1], [0, 0]], ids=str)
def test_rows(rows, actuated):
    rng = np.random.default_rng(len(rows))
    x, ends = [], []
    for s, d in enumerate(rows):
        x.append(rng.uniform(-0.4, 0.4, (64, 3)) + np.array([2.0 * s, 0.0, 0.0]))
        ends += [(64 * s, 64 * s + 1 + j) for j in range(d)]
    _same(np.concatenate(x), np.array(ends, np.int32).reshape(-1, 2), 0.45 + 0.1 * (np.arange(len(ends)) % 3), actuated)


@pytest.mark.parametrize("n", [1, 63, 65, 16383, 16384, 16385])
def test_sizes(n):
    rng = np.random.default_rng(n)
    x = np.stack([np.arange(n) * 0.5, np.zeros(n), 0.1 * rng.uniform(-1, 1, n)], 1) + 0.01 * rng.normal(size=(n, 3))
    ends = np.array([(i, i + d) for d in (1, 2, 5) for i in range(0, max(0, n - d))], np.int32).reshape(-1, 2)
    _same(x, ends, np.full(len(ends), 0.6), False)
