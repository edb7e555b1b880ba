"""The gradient of a body that has actuation groups but no spring in any of them: every sensitivity is
zero and the rest is the passive body's, to the rounding of the forms' sums.  With one, two and four
lanes per mass, and for groups that some workgroups' springs are members of and others' are not."""
import numpy as np
import pytest

from paper_2207_09334_amd import cronos as CR

pytestmark = pytest.mark.gpu


def _body():
    rng = np.random.default_rng(11)
    x = rng.uniform(0.0, 1.0, (300, 3))
    ends = np.array([(i, i + d) for d in (1, 7, 30) for i in range(300 - d)], np.int32)
    return x, ends, rng.normal(size=x.shape)


def _gradient(lanes, group, n_groups=5):
    x, ends, w = _body()
    kw = {} if group is None else dict(group=group.astype(np.int16), n_groups=n_groups)
    sim = CR.cronos_create(x, np.full(len(x), 0.1), ends, np.full(len(ends), 500.0), np.full(len(ends), 0.5), dt=1e-4,
                           block_masses=64, lanes_per_mass=lanes, flags=CR.ALLOW_UNSTABLE, **kw)
    if group is not None:
        CR.cronos_set_actuation(sim, np.full(n_groups, 0.7), np.full(n_groups, 0.3), 2.0)
    loss = CR.cronos_rollout(sim, 5, 2, w)
    out = [np.float64(loss)] + [np.asarray(g) for g in CR.cronos_rollout_backward(sim, want_state=True)]
    sim.close()
    return out


@pytest.mark.parametrize("lanes", [1, 2, 4])
def test_no_spring_in_any_group(lanes):
    ends = _body()[1]
    a, b = _gradient(lanes, np.full(len(ends), -1)), _gradient(lanes, None)
    assert a[1].shape == a[2].shape == (5,) and not a[1].any() and not a[2].any()
    # five steps of at most 6 springs a mass: 5 * 8 * 2^-24 of the largest
    for p, q in ((a[0], b[0]), (a[3], b[3]), (a[4], b[4])):
        assert np.abs(q).max() > 0 and np.abs(p - q).max() <= 40 * 2.0 ** -24 * np.abs(q).max()


@pytest.mark.parametrize("lanes", [1, 2, 4])
def test_members_in_one_workgroup_only(lanes):
    """One spring is a member; its group's gradient is that of the same body with the group's number moved
    up by one, bit for bit: the same sum."""
    ends = _body()[1]
    group = np.full(len(ends), -1)
    group[17] = 2
    a, b = _gradient(lanes, group), _gradient(lanes, group + (group >= 0), n_groups=6)
    assert np.flatnonzero(a[2]).tolist() == [2] and np.flatnonzero(b[2]).tolist() == [3]
    assert a[1][2] == b[1][3] and a[2][2] == b[2][3] and np.array_equal(a[3], b[3]) and np.isfinite(a[3]).all()
