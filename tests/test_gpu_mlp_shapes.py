"""The network's kernels at the edges of their tiles: widths below, at and beside multiples of 32, 64
and 128, output layers narrow (a wavefront per 16 rows) and wide, row counts from 1 to several tiles
and splits, pre-activations small and far out (both ways of erf).  Against the FP64 oracle that
rounds to BF16 where the device stores BF16, at the bars of the surrogate tests."""
import numpy as np
import pytest

import workloads as W
from oracle import mlp as M
from paper_2207_09334_amd import cronos as CR
from tests.gpu_common import say
from tests.test_gpu_surrogate import G_TOL, Y_TOL, _elem, _rel

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1, 1, 1), (7, 33, 70, 130, 3), (96, 64, 128, 192, 16), (96, 100, 36, 65, 17), (33, 256, 512, 96, 70),
         (96, 768, 768, 768, 3)]


def _case(sizes, rows, scale, seed):
    rng = np.random.default_rng(seed)
    params = [scale * p + 0.05 * rng.normal(size=p.shape) for p in W.mlp_init(seed, sizes)]
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    return params, f32(rng.normal(size=(rows, sizes[0]))), f32(rng.normal(size=(rows, sizes[4])))


@pytest.mark.parametrize("scale", [1.0, 4.0])
@pytest.mark.parametrize("rows", [1, 63, 65, 1030])
@pytest.mark.parametrize("sizes", SIZES)
def test_forward_and_gradients(sizes, rows, scale):
    say(f"case: {sizes}, {rows} rows, weights x {scale}")
    params, X, T = _case(sizes, rows, scale, rows)
    net = CR.cronos_mlp_create(params, sizes=sizes, max_rows=rows)
    y = CR.cronos_mlp_forward(net, X)
    ref, _ = M.forward(params, X, storage="bf16")
    assert _rel(y, ref) <= Y_TOL
    loss, g = CR.cronos_mlp_loss_grad(net, X, T)
    lo, go = M.loss_and_grad(params, X, T, storage="bf16")
    assert loss == pytest.approx(lo, rel=1e-4)
    for a, b in zip(g, go):
        assert _rel(a, b) <= G_TOL
    # the forward that the gradients ran on kept more of itself, with the same result
    assert np.array_equal(y, CR.cronos_mlp_forward(net, X))
    net.close()


@pytest.mark.parametrize("rows", [5700, 6144])
def test_wide_tiles(rows):
    """Enough rows for the 128 x 128 tiles of the forward products: the same bits as in small chunks."""
    sizes = (96, 768, 704, 768, 3)
    params, X, T = _case(sizes, rows, 2.0, 5)
    y = [CR.cronos_mlp_forward(CR.cronos_mlp_create(params, sizes=sizes, max_rows=m), X) for m in (rows, 640)]
    assert np.array_equal(y[0], y[1])
    ref, _ = M.forward(params, X, storage="bf16")
    assert _rel(y[0], ref) <= Y_TOL and _elem(y[0], ref, axis=0) <= Y_TOL * 2


@pytest.mark.parametrize("sizes", SIZES)
def test_adam_and_the_weights_it_leaves(sizes):
    """One Adam step on every layer shape, and a forward through the weights it leaves (both BF16
    copies of them: the forward reads one, the gradients the other)."""
    params, X, T = _case(sizes, 200, 1.0, 9)
    net = CR.cronos_mlp_create(params, sizes=sizes, max_rows=600)
    _, g = CR.cronos_mlp_loss_grad(net, X, T)
    CR.cronos_mlp_adam(net, lr=1e-2)
    after = CR.cronos_mlp_get_params(net)
    ref = [np.asarray(p, np.float32).astype(np.float64) for p in params]
    M.adam_step(ref, g, [np.zeros_like(p) for p in ref], [np.zeros_like(p) for p in ref], 1, lr=1e-2)
    for a, r in zip(after, ref):
        np.testing.assert_allclose(a, r, rtol=1e-5, atol=1e-6)
    y = CR.cronos_mlp_forward(net, X)
    assert _rel(y, M.forward(after, X, storage="bf16")[0]) <= Y_TOL
    _, g = CR.cronos_mlp_loss_grad(net, X, T)
    _, go = M.loss_and_grad(after, X, T, storage="bf16")
    for a, b in zip(g, go):
        assert _rel(a, b) <= G_TOL
    net.close()


def test_training_loss_is_the_last_epochs():
    """The loss of the last epoch's minibatches (a short last one among them) with the weights held:
    the rows' mean loss, whatever their order."""
    sizes = (20, 64, 64, 64, 3)
    params, X, T = _case(sizes, 1000, 1.0, 3)
    net = CR.cronos_mlp_create(params, sizes=sizes, max_rows=300)
    loss = CR.cronos_mlp_train(net, X, T, batch=300, epochs=3, lr=0.0, lr_final=0.0, seed=7)
    y, _ = M.forward(params, X, storage="bf16")
    assert loss == pytest.approx(float(((y - T) ** 2).mean()), rel=1e-4)
    net.close()
