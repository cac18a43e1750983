"""The surrogate network's loss past 512 chunks of 16 samples, where a thread adds
terms of several chunks (needs an MI355X).

With zero output weights the network returns 0, and with targets that are powers
of two and a sum of weights that is one, every term m t^2 / (2 sum m) is exact in
FP32.  The first 8,192 rows (the first chunk of each workgroup) have terms 2^26
times those of the others: an FP32 sum over a workgroup's chunks loses all of the
small ones, 1.2e-7 (2^15 rows) to 1.9e-6 (2^20) of the loss.  FP64 sums, on the
GPU and here, are exact to their round-off, 2^20 additions of at most 2^-53.
"""
import numpy as np
import pytest
import torch

from paper_1306_6445_amd import lbm, surrogate as SG

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [2 ** 13, 2 ** 15, 2 ** 20])
@pytest.mark.parametrize("train", [False, True])
def test_loss_of_many_chunks_is_summed_in_fp64(rows, train):
    params = SG.init_params(3)
    params[-(3 * 64 + 3):] = 0.0
    t = np.full((rows, 3), 2.0 ** -13, dtype=np.float32)
    t[:8192] = 1.0
    m = np.ones((rows, 3), dtype=np.float32)
    m[:, 2] = 0.0
    x = np.random.default_rng(0).uniform(-1, 1, (rows, 3)).astype(np.float32)
    x, tt, mm = (torch.from_numpy(v).to("cuda") for v in (x, t, m))
    with lbm.Mlp(params, max_batch=rows) as net:
        loss = net.train(x, tt, mm, steps=1, lr=1e-3) if train else net.loss_grad(x, tt, mm)[0]
    t, m = t.astype(np.float64), m.astype(np.float64)
    want = np.sum(m * t * t) / (2 * np.sum(m))
    assert abs(loss - want) <= 2.0 ** 20 * 2.0 ** -53 * want
