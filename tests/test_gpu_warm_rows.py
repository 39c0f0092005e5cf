"""GPU parity of the network's small products, which take a wave per 16 rows of a tile, at the
edges of that split and on both sides of the line to a wave per tile; and of one to four rows
with fewer values than the matrix-vector kernel has K groups.

Bar as in test_gpu_warm.py: FP32 products over at most 700 terms of random sign
(sqrt(700) 2^-24 = 2e-6, inside 1e-5).
"""
import numpy as np
import pytest
import torch

from oracle import mlp as om
from paper_1702_02241_amd import torch_api as T

from gpu_common import device, rel
from test_gpu_warm import _net_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,din,dh,mu,nv,k", [
    (16, 300, 16, 20, 5, 3),      # one row tile full, the others empty
    (17, 301, 17, 21, 5, 3),      # one row past it; every length odd
    (63, 64, 63, 16, 4, 2),       # last row tile one short
    (81, 130, 40, 30, 7, 5),      # two tiles of rows, the second with two row tiles
    (128, 16, 128, 64, 7, 9),     # K of one block, K of eight; weight gradients with a K of eight
    (5, 700, 130, 3200, 14, 20),  # grad W2 on the other side of the line (3,015 tiles)
    (3, 64, 8, 40, 9, 4),         # few rows, K below the K groups
    (1, 64, 31, 40, 9, 4),        # one row, the same
    (2, 40, 32, 40, 9, 4),        # few rows, K equal to them
])
def test_network_matches_oracle(B, din, dh, mu, nv, k):
    dev = device()
    x, W1, b1, W2, b2, TU, TV = _net_case(B, din, dh, mu, nv, k, seed=5 * B + k)
    net = T.WarmNet(din, dh, mu, nv, k, max_batch=B, seed=1)
    net.set_params(W1, b1, W2, b2)
    d = [a.astype(np.float64) for a in (x, W1, b1, W2, b2, TU, TV)]
    xd, TUd, TVd = (torch.from_numpy(a).to(dev) for a in (x, TU, TV))
    y = net.forward(xd)
    loss = net.loss_grad(xd, TUd, TVd)
    _, _, yr = om.forward(*d[:5])
    lr, dW1, db1, dW2, db2 = om.loss_grad(d[0], np.matmul(d[5], d[6].transpose(0, 2, 1)), *d[1:5], mu, nv, k)
    g = net.grads()
    errs = [rel(y.cpu().numpy(), yr), abs(loss.item() - lr) / abs(lr), rel(g[0].reshape(din, dh), dW1), rel(g[1], db1),
            rel(g[2].reshape(dh, -1), dW2), rel(g[3], db2)]
    print(f"[mlp rows B={B} {din}-{dh}-{(mu + nv) * k} k={k}] " + " ".join(f"{e:.1e}" for e in errs), flush=True)
    assert max(errs) <= 1e-5
    net.close()
