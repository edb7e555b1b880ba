"""The surrogate trains the network of the width it was asked for, and a network is created only from at least
as many parameters as its layers hold."""
import numpy as np
import pytest

import workloads as W
from paper_2207_09334_amd import cronos as CR, surrogate as SG


@pytest.mark.parametrize("width", [64, 256, 768])
def test_network_has_the_width_asked_for(monkeypatch, width):
    made = {}

    def create(params, sizes=(96, 256, 256, 256, 3), max_rows=4096, device=0, stream=None):
        made.update(sizes=tuple(sizes), shapes=[np.shape(p) for p in params])

    monkeypatch.setattr(CR, "cronos_mlp_create", create)
    monkeypatch.setattr(CR, "cronos_mlp_train", lambda *a, **k: 0.0)
    rng = np.random.default_rng(0)
    SG.Surrogate(rng.normal(size=(8, 96)), rng.normal(size=(8, 3)), width=width)
    assert made["sizes"] == (96, width, width, width, 3)
    assert made["shapes"][::2] == [(96, width), (width, width), (width, width), (width, 3)]


@pytest.mark.parametrize("given, sizes", [((96, 256, 256, 256, 3), (96, 768, 768, 768, 3)), ((4, 5, 6, 7, 2), (4, 5, 6, 7, 3)),
                                          ((4, 5, 6, 7, 2), (4, 5, 6, 7))])
def test_too_few_parameters_are_refused(given, sizes):
    with pytest.raises(CR.CronosError):
        CR.cronos_mlp_create(W.mlp_init(1, given), sizes=sizes)
