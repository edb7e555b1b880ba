"""The gradient of a few steps with one, two and four lanes per mass, on bodies whose slices hold every
number of entry rows from none to several groups of the lanes' rows: the forms differ only in the
order of the sums over a mass's springs, so they agree to FP32 rounding, actuated and passive."""
import numpy as np
import pytest

from paper_2207_09334_amd import cronos as CR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("actuated", [False, True])
@pytest.mark.parametrize("rows", [list(range(0, 20)), [0, 0], [1], [33, 34], [63]], ids=str)
def test_lanes_agree(rows, actuated):
    rng = np.random.default_rng(len(rows))
    x, ends, at = [], [], 0
    for d in rows:
        x.append(rng.uniform(0.1, 0.9, (64, 3)) + np.array([2.0 * len(x), 0.0, 0.0]))
        ends += [(at, at + 1 + j) for j in range(d)]
        at += 64
    x, ends = np.concatenate(x), np.array(ends, np.int32).reshape(-1, 2)
    s = len(ends)
    kw = dict(dt=1e-4, damping=1e-3, flags=CR.ALLOW_UNSTABLE)
    groups = (np.arange(s) % 7 - 1).astype(np.int16)
    if actuated and s:
        kw.update(group=groups, n_groups=6)
    w = rng.normal(size=x.shape)
    out = []
    for lanes in (1, 2, 4):
        sim = CR.cronos_create(x, np.full(len(x), 0.1), ends, np.full(s, 500.0),
                               np.full(s, 0.5) + 0.1 * (np.arange(s) % 3), lanes_per_mass=lanes, **kw)
        if actuated and s:
            CR.cronos_set_actuation(sim, np.linspace(0.1, 3.0, 6), np.linspace(0.0, 0.3, 6), 2.0)
        loss = CR.cronos_rollout(sim, 5, 2, w)
        out.append([np.float64(loss)] + [np.asarray(g) for g in CR.cronos_rollout_backward(sim, want_state=True)])
        assert s == 0 or CR.cronos_launch_config(sim)["lanes_per_mass"] == lanes
        sim.close()
    # five steps of up to 63 springs a mass, each sum of at most 63 FP32 terms: 5 * 63 * 2^-24 of the largest
    tol = 5 * 64 * 2.0 ** -24
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.all(np.isfinite(a)) and a.shape == b.shape
            if a.size:
                assert np.abs(a - b).max() <= tol * max(np.abs(a).max(), 1e-30)


def test_sums_by_workgroup_and_by_entry_agree():
    """Six groups numbered densely (their sums are held by each workgroup) and spread over 600 numbers (too
    wide a range for that: one sum per entry) have the same gradient.  Both add the same FP64 terms,
    under 2^12 of them, in another order: 2^12 * 2^-53 of the terms' sum, which is under 100 times
    the largest component here."""
    rng = np.random.default_rng(5)
    x = rng.uniform(0.0, 1.0, (300, 3))
    ends = np.array([(i, j) for i in range(300) for j in (i + 1, i + 7, i + 30) if j < 300], np.int32)
    s = len(ends)
    groups = np.arange(s) % 7 - 1
    phase, amp, w = np.linspace(0.1, 3.0, 6), np.linspace(0.1, 0.3, 6), rng.normal(size=x.shape)
    for lanes in (1, 2, 4):
        out = []
        for step in (1, 100):
            at = np.arange(6) * step
            sim = CR.cronos_create(x, np.full(300, 0.1), ends, np.full(s, 500.0), np.full(s, 0.5), lanes_per_mass=lanes,
                                   group=np.where(groups < 0, -1, groups * step).astype(np.int16), n_groups=5 * step + 1,
                                   dt=1e-4, flags=CR.ALLOW_UNSTABLE)
            ph, am = np.zeros(5 * step + 1), np.zeros(5 * step + 1)
            ph[at], am[at] = phase, amp
            CR.cronos_set_actuation(sim, ph, am, 2.0)
            loss = CR.cronos_rollout(sim, 4, 2, w)
            g = CR.cronos_rollout_backward(sim, want_state=True)
            out.append((loss, g[0][at], g[1][at], g[2], g[3]))
            rest = np.setdiff1d(np.arange(5 * step + 1), at)
            assert not g[0][rest].any() and not g[1][rest].any()
            sim.close()
        a, b = out
        assert a[0] == b[0] and np.array_equal(a[3], b[3]) and np.array_equal(a[4], b[4])
        for p, q in zip(a[1:3], b[1:3]):
            assert np.abs(p).max() > 0 and np.abs(p - q).max() <= 2.0 ** -41 * 100 * np.abs(p).max()
