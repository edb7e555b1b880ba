"""Where the reverse step sums each group's sensitivities follows from the body's size, its rows and the groups of
a workgroup: on either side of every line of that rule, six groups numbered densely have the gradient of the
same six spread over 600 numbers (a range too wide for anything but a sum per entry)."""
import numpy as np
import pytest

from paper_2207_09334_amd import cronos as CR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes", [1, 2, 4])
@pytest.mark.parametrize("n, degree", [(300, 24), (300, 18), (300, 6), (8191, 24), (8191, 6), (8192, 6), (8192, 4),
                                       (32767, 4), (32768, 4), (32768, 2)])
def test_dense_and_spread_numbers_agree(n, degree, lanes):
    rng = np.random.default_rng(n + degree)
    x = np.stack([0.3 * np.arange(n), np.zeros(n), np.zeros(n)], 1) + rng.uniform(0.0, 0.2, (n, 3))
    ends = np.concatenate([np.stack([np.arange(n - d), np.arange(d, n)], 1) for d in range(1, degree // 2 + 1)]).astype(np.int32)
    s = len(ends)
    groups = np.arange(s) % 7 - 1
    phase, amp, w = np.linspace(0.1, 3.0, 6), np.linspace(0.1, 0.3, 6), rng.normal(size=x.shape)
    out = []
    for step in (1, 100):
        at = np.arange(6) * step
        sim = CR.cronos_create(x, np.full(n, 0.1), ends, np.full(s, 500.0), np.full(s, 0.5), lanes_per_mass=lanes,
                               block_masses=64, group=np.where(groups < 0, -1, groups * step).astype(np.int16),
                               n_groups=5 * step + 1, dt=1e-4, flags=CR.ALLOW_UNSTABLE)
        ph, am = np.zeros(5 * step + 1), np.zeros(5 * step + 1)
        ph[at], am[at] = phase, amp
        CR.cronos_set_actuation(sim, ph, am, 2.0)
        loss = CR.cronos_rollout(sim, 4, 2, w)
        g = CR.cronos_rollout_backward(sim, want_state=True)
        out.append((loss, g[0][at], g[1][at], g[2], g[3]))
        sim.close()
    a, b = out
    assert a[0] == b[0] and np.array_equal(a[3], b[3]) and np.array_equal(a[4], b[4])
    # the same FP64 terms in another order, under 2^17 of them: 2^17 * 2^-53 of their magnitudes' sum, which is
    # under 1000 times the largest component
    for p, q in zip(a[1:3], b[1:3]):
        assert np.abs(p).max() > 0 and np.abs(p - q).max() <= 2.0 ** -36 * 1000 * np.abs(p).max()
