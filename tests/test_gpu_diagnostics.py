"""Diagnostics of bodies with every remainder of chunks per lane of the per-body sum and of entry rows per
batch, against the same sums in FP64 NumPy from the state read back."""
import numpy as np
import pytest

from paper_2207_09334_amd import cronos as CR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [0, 1, 2, 3, 4, 7])
@pytest.mark.parametrize("n", [1, 64, 65, 63 * 64, 64 * 64 + 1, 130 * 64 + 5])
def test_sums(n, degree):
    rng = np.random.default_rng(n + degree)
    x, v, m = rng.uniform(-1, 1, (n, 3)), rng.normal(size=(n, 3)), np.float64(np.float32(0.25)) * np.ones(n)
    ends = np.array([(i, i + d) for d in range(1, degree + 1) for i in range(0, n - d, 2)], np.int32).reshape(-1, 2)
    rest = np.full(len(ends), 0.5)
    cut = [0, n // 3, n] if n > 2 and degree == 0 else [0, n]
    sim = CR.cronos_create(x, m, ends, np.full(len(ends), 8.0), rest, v0=v, dt=1e-4, block_masses=64,
                           flags=CR.NO_SHIFT | CR.ALLOW_UNSTABLE, body_offset=cut if len(cut) > 2 else None)
    x, v, _ = CR.cronos_read_state(sim)
    for b, (lo, hi) in enumerate(zip(cut, cut[1:])):
        d = CR.cronos_diagnostics(sim)[b]
        xb, vb, mb = x[lo:hi], v[lo:hi], m[lo:hi]
        length = np.linalg.norm(x[ends[:, 1]] - x[ends[:, 0]], axis=1) if len(ends) else np.zeros(0)
        # sums of at most 2^16 FP64 terms, each right to a few units of 2^-53: 2^16 * 2^-53 of the terms' magnitudes
        near = lambda got, terms: np.all(np.abs(np.asarray(got) - terms.sum(0)) <= 2.0 ** -36 * np.abs(terms).sum(0))
        assert near(d["ke"], 0.5 * mb * (vb * vb).sum(1))
        assert near(d["pe_spring"], 0.5 * 8.0 * (length - 0.5) ** 2)
        assert near(
            d["pe_grav"], -mb * float(np.float32(-9.81)) * xb[:, 2])
        assert near(d["p"], mb[:, None] * vb) and near(np.asarray(d["com"]) * mb.sum(), mb[:, None] * xb)
        assert near(d["mass"], mb)
        assert np.array_equal(d["bbox_min"], xb.min(0)) and np.array_equal(d["bbox_max"], xb.max(0))
    sim.close()
