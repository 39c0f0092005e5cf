"""GPU parity of the thin Gram matrices (certificate, preconditioner) at the edges of their
kernel: ranks one block of 16 columns holds and two, rows that do not fill a group of four,
fewer groups than waves and more than one pass.

Singular values of U V^T come from FP64 sums of exact products of FP32 entries (1e-6 covers
the square root of the smallest over the largest, 1e-3 here); T1..T3 carry the FP32 gradient
rows: 1e-3 of the larger of the term and one, the certificate tests' bar.  A preconditioned
step reports the objective at the factors it returns (1e-5).
"""
import numpy as np
import pytest
import torch

from oracle import certificate as ce
from oracle import objective as ob
from paper_1702_02241_amd import synth
from paper_1702_02241_amd import torch_api as T

from gpu_common import device, f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(33, 17, 1), (70, 45, 10), (131, 66, 16), (1025, 79, 17), (4099, 65, 20),
                                   (40000, 64, 32)])
def test_certificate_and_preconditioned_step(m, n, k):
    p = synth.gaussian_rpca(m=m, n=n, r=min(5, k), k=k, seed=m + k)
    U, V = synth.random_factors(m, n, k, 11 + k, scale=0.5)
    dev = device()
    ctx = T.Context(m, n, k, p.lam_s, p.lam_l)
    Xcm = T.to_device_X(p.X, dev)
    Ud, Vd = T.to_device_factor(U, dev), T.to_device_factor(V, dev)
    c = ctx.certificate(Xcm, Ud, Vd)
    o = ce.certificate(f32(U), f32(V), f32(p.X), p.lam_s, p.lam_l, tau=1e-6)
    s = np.linalg.svd(np.linalg.qr(f32(U))[1] @ np.linalg.qr(f32(V))[1].T, compute_uv=False)
    es = np.max(np.abs(np.array(c.sigma[:k]) - s)) / s[0]
    print(f"[rows gram {m}x{n} k={k}] sigma {es:.1e} T ({c.T1:.5g},{c.T2:.5g},{c.T3:.5g}) "
          f"oracle ({o['T1']:.5g},{o['T2']:.5g},{o['T3']:.5g})")
    assert c.r == o["r"] and es <= 1e-6
    for key in ("T1", "T2", "T3"):
        assert abs(getattr(c, key) - o[key]) <= 1e-3 * max(o[key], 1.0), key
    rc, info = ctx.solve(Xcm, Ud, Vd, precond=1, max_iter=1)
    torch.cuda.synchronize()
    f = ob.objgrad(Ud.cpu().numpy().astype(np.float64), Vd.cpu().numpy().astype(np.float64), f32(p.X), p.lam_s,
                   p.lam_l)[0]
    assert abs(info.f - f) <= 1e-5 * abs(f)
    ctx.close()
