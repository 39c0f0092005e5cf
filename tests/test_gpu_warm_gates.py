"""The gates of the network's training step do not depend on the batch size.

A hidden unit's gate is the sign of its input as FP32 sums it, through K in order.  Here every
unit's input is 2^24 + 1 - 2^24 with the last term 32 entries after the first: 0 in K order
(2^24 + 1 rounds to 2^24), 1 if the large terms meet first.  So no unit is on, and grad W1 is
zero, for batches that other products of few rows would take as well as for larger ones.
"""
import numpy as np
import pytest
import torch

from paper_1702_02241_amd import torch_api as T

from gpu_common import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 17])
def test_gates_follow_the_sum_in_order(batch):
    d_in, d_h, mu, nv, k = 64, 24, 10, 6, 2
    net = T.WarmNet(d_in, d_h, mu, nv, k, max_batch=batch)
    W1 = np.zeros((d_in, d_h), np.float32)
    W1[0], W1[1], W1[32] = 2.0 ** 24, 1.0, -(2.0 ** 24)
    rng = np.random.default_rng(0)
    W2 = rng.standard_normal((d_h, (mu + nv) * k)).astype(np.float32)
    net.set_params(W1, np.zeros(d_h, np.float32), W2, np.ones((mu + nv) * k, np.float32))
    dev = device()
    x = torch.ones(batch, d_in, device=dev)
    TU, TV = torch.zeros(batch, mu, k, device=dev), torch.zeros(batch, nv, k, device=dev)
    loss = net.loss_grad(x, TU, TV)
    torch.cuda.synchronize()
    gW1, gb1, gW2, gb2 = [np.asarray(g) for g in net.grads()]
    print(f"[gates batch={batch}] loss {float(loss):.6g} |gW1| {np.abs(gW1).max()} |gb2| {np.abs(gb2).max()}", flush=True)
    assert np.abs(gb2).max() > 0  # the output layer learns: only the gates are off
    assert not gW1.any() and not gb1.any() and not gW2.any()
    net.close()
