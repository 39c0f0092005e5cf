"""GPU parity of the warm-start kernels at the edges of their tiles and dispatch rules.

* the network's products: one to four rows take the matrix-vector kernel (row lengths
  divisible by four or not, one K range or several), more rows the 64 x 64 tiles (ragged
  rows, columns and K; K of at most eight blocks in one wave or split over waves and
  workgroups);
* the loss: k up to 16 and up to 32, one row chunk or several, ragged last rows;
* the window statistics: 4 x 4 pooling from 16-byte aligned and from unaligned data, other
  pooling factors, more and fewer frames than frame groups.

Bars as in test_gpu_warm.py: FP32 products with FP32 accumulation over at most 2,600 terms
of random sign (sqrt(2600) 2^-24 = 3e-6, inside 1e-5); means and deviations in FP64, rounded
once (1e-6).
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
    (1, 2600, 64, 40, 8, 4),     # matrix-vector, K split over workgroups, 16-byte rows
    (2, 130, 33, 7, 4, 3),       # matrix-vector, rows of odd length
    (4, 513, 36, 9, 3, 5),       # most rows of the matrix-vector kernel, K one past a staging slice
    (5, 129, 65, 13, 4, 3),      # fewest rows of the tiles, one past a tile and past eight K blocks
    (65, 128, 64, 16, 16, 2),    # two row tiles, K exactly eight blocks
    (130, 31, 70, 300, 21, 17),  # rank above 16, batch K beyond eight blocks, several row chunks
    (9, 40, 20, 1030, 3, 32),    # largest rank, chunks of 256 rows with a ragged last one
])
def test_network_matches_oracle_at_the_edges(B, din, dh, mu, nv, k):
    dev = device()
    x, W1, b1, W2, b2, TU, TV = _net_case(B, din, dh, mu, nv, k, seed=3 * B + k)
    net = T.WarmNet(din, dh, mu, nv, k, max_batch=B, seed=1)
    net.set_params(W1, b1, W2, b2)
    d = [a.astype(np.float64) for a in (x, W1, b1, W2, b2, TU, TV)]
    xd, TUd, TVd = (torch.from_numpy(a).to(dev) for a in (x, TU, TV))
    y = net.forward(xd)
    loss = net.loss_grad(xd, TUd, TVd)
    _, _, yr = om.forward(*d[:5])
    T_dense = np.matmul(d[5], d[6].transpose(0, 2, 1))
    lr, dW1, db1, dW2, db2 = om.loss_grad(d[0], T_dense, *d[1:5], mu, nv, k)
    g = net.grads()
    errs = [rel(y.cpu().numpy(), yr), abs(loss.item() - lr) / abs(lr), rel(g[0].reshape(din, dh), dW1), rel(g[1], db1),
            rel(g[2].reshape(dh, -1), dW2), rel(g[3], db2)]
    print(f"[mlp edges B={B} {din}-{dh}-{(mu + nv) * k} k={k}] " + " ".join(f"{e:.1e}" for e in errs))
    assert max(errs) <= 1e-5
    net.close()


@pytest.mark.parametrize("W,H,f,frames,offset", [(132, 8, 4, 33, 0), (132, 8, 4, 33, 1), (20, 12, 4, 1, 0), (35, 21, 7, 40, 0),
                                                 (6, 4, 2, 3, 3)])
def test_window_features_match_oracle_at_the_edges(W, H, f, frames, offset):
    dev = device()
    rng = np.random.default_rng(W + f)
    X = rng.uniform(size=(frames, W * H)).astype(np.float32)
    buf = torch.zeros(frames * W * H + offset, dtype=torch.float32, device=dev)
    Xcm = buf[offset:].view(frames, W * H)  # offset: 4-byte but not 16-byte aligned
    Xcm.copy_(torch.from_numpy(X))
    feat = T.window_features(Xcm, W, H, frames, f).cpu().numpy()
    ref = om.window_features(X.T.astype(np.float64), W, H, f)
    assert rel(feat, ref) <= 1e-6 and float(np.max(np.abs(feat - ref))) <= 1e-6
