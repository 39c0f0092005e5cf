"""The preconditioner's Gram matrices, through what depends on their values: the first step.

In the variables A = U P_U^{-1}, B = V P_V^{-1} the first L-BFGS step goes along the negative
gradient, which in the plain variables is -(gU (V^T V + lam_L I)^{-1}, gV (U^T U + lam_L I)^{-1}):
one step length for both factors.  Compared with the FP64 oracle's gradient and Gram matrices at
ranks of one block of 16 columns and two, and rows that do not fill the kernel's groups.

Bound: the change of variables and back rounds the factors (6e-8 sqrt(k) cond(P), cond below 10
for these factors: 3e-6 of the factor), the gradient is within 1e-5 of itself; 1e-4 of the step
leaves a factor for the conditioning of the inverse.
"""
import numpy as np
import pytest
import torch

from oracle import objective as ob
from paper_1702_02241_amd import synth
from paper_1702_02241_amd import torch_api as T

from gpu_common import device, f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(33, 17, 1), (70, 45, 10), (131, 66, 16), (1025, 79, 17), (259, 65, 20), (301, 64, 32)])
def test_first_preconditioned_step(m, n, k):
    p = synth.gaussian_rpca(m=m, n=n, r=min(5, k), k=k, seed=m + k)
    U, V = synth.random_factors(m, n, k, 21 + k, scale=0.5)
    U, V = f32(U), f32(V)
    dev = device()
    ctx = T.Context(m, n, k, p.lam_s, p.lam_l)
    Ud, Vd = T.to_device_factor(U, dev), T.to_device_factor(V, dev)
    _, info = ctx.solve(T.to_device_X(p.X, dev), Ud, Vd, precond=1, max_iter=1, gtol=0.0, ftol=0.0, certify=0)
    torch.cuda.synchronize()
    ctx.close()
    _, gU, gV = ob.objgrad(U, V, f32(p.X), p.lam_s, p.lam_l)
    I = np.eye(k)
    D = np.concatenate([-gU @ np.linalg.inv(V.T @ V + p.lam_l * I), -gV @ np.linalg.inv(U.T @ U + p.lam_l * I)])
    S = np.concatenate([Ud.cpu().numpy().astype(np.float64) - U, Vd.cpu().numpy().astype(np.float64) - V])
    alpha = np.sum(S * D) / np.sum(D * D)
    off = np.linalg.norm(S - alpha * D)
    nx = np.linalg.norm(np.concatenate([U, V]))
    print(f"[precond step {m}x{n} k={k}] alpha {alpha:.4g} step {np.linalg.norm(S) / nx:.2e} off {off / np.linalg.norm(S):.2e}",
          flush=True)
    assert info.iters == 1 and alpha > 0
    assert off <= 1e-4 * np.linalg.norm(S) + 3e-6 * nx
