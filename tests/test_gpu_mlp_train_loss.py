"""The loss that training reports for its last epoch, for output layers on either side of every change in
how many partial sums a minibatch leaves (16 columns: one per 16 rows; above, one per 64 x 64 tile, up
to 64 tiles across), with several minibatches, the last one short.  The weights are held, so it is the
rows' mean loss whatever their order."""
import pytest

from oracle import mlp as M
from paper_2207_09334_amd import cronos as CR
from tests.gpu_common import say
from tests.test_gpu_mlp_shapes import _case
from tests.test_gpu_surrogate import Y_TOL, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows, batch", [(1000, 300), (300, 1000), (130, 1), (2100, 1000)])
@pytest.mark.parametrize("n_out", [3, 16, 17, 64, 65, 70, 256, 257, 600, 1024, 4096])
def test_last_epochs_loss(n_out, rows, batch):
    say(f"case: {n_out} outputs, {rows} rows, minibatches of {batch}")
    sizes = (20, 64, 40, 64, n_out)
    params, X, T = _case(sizes, rows, 1.0, n_out)
    net = CR.cronos_mlp_create(params, sizes=sizes, max_rows=max(batch, 1))
    loss = CR.cronos_mlp_train(net, X, T, batch=batch, epochs=2, lr=0.0, lr_final=0.0, seed=7)
    y, _ = M.forward(params, X, storage="bf16")
    assert loss == pytest.approx(float(((y - T) ** 2).mean()), rel=1e-4)
    # the weights that it left are still those given
    out = CR.cronos_mlp_forward(net, X[:64])
    assert _rel(out, y[:64]) <= Y_TOL
    net.close()
