"""Loss and gradient of the surrogate network at the edges of its chunks (needs
an MI355X): batches of one sample, one short of and one past a chunk of 16, and
past 512 chunks, where workgroups take several, against the FP64 network.

Tolerance: a gradient entry sums n products of order 1 / (3 n) in FP32, chunks
in order and then the slots, so its rounding is below (16 + 3 n / 16) unit
round-offs of the sum of magnitudes; n = 9,000 gives 1.0e-4 of the largest
entry at most, and 2e-5 is its random-walk size with a margin of ten.
"""
import numpy as np
import pytest

from oracle import mlp as OM
from paper_1306_6445_amd import lbm, surrogate as SG

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 8192, 9000])
def test_loss_and_gradient_at_chunk_edges(n):
    rng = np.random.default_rng(n)
    params = SG.init_params(n)
    x = rng.uniform(-1, 1, (n, 3)).astype(np.float32)
    t = rng.uniform(-1, 1, (n, 3)).astype(np.float32)
    m = rng.uniform(0.5, 1.0, (n, 3)).astype(np.float32)
    with lbm.Mlp(params, max_batch=n) as net:
        loss, grad = net.loss_grad(x, t, m)
        y = net.forward(x)
    want_loss, want_grad = OM.loss_and_grad(params.astype(np.float64), x.astype(np.float64), t.astype(np.float64),
                                            m.astype(np.float64))
    want_y = OM.forward(params.astype(np.float64), x.astype(np.float64))
    want_y = want_y[0] if isinstance(want_y, tuple) else want_y
    assert abs(loss - want_loss) <= 2e-5 * abs(want_loss)
    assert np.max(np.abs(grad - want_grad)) <= 2e-5 * np.max(np.abs(want_grad))
    assert np.max(np.abs(y - want_y)) <= 2e-5
