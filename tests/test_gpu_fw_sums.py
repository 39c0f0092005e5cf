"""Frank-Wolfe: the bilinear sums of the exact line search are sums in 64 bits.

Every row of L is the same and L - X is past the threshold everywhere, so G is constant:
with n = 256 columns v = 1/16, y_i = sum_j G_ij v_j = 1 and sum_j v_j^2 = 1 exactly in FP32,
and u^T L v = m z / sigma, z = sum_j l_j / 16, whose products are exact.  The step length then
follows from the reported phi and sigma in 64 bits; a rounding of z in FP32, common to all rows,
would show in it (2e-8).  m odd: the pass that reads single rows.
"""
import numpy as np
import pytest
import torch

from paper_1702_02241_amd import torch_api as T

from gpu_common import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,seed", [(1001, 0), (1001, 1), (4099, 2), (77, 3)])
def test_step_length_from_sums_in_64_bits(m, seed):
    n, lam_s, lam_l = 256, 2.0 ** -4, 0.3 * (2.0 ** -4) * (256 * m) ** 0.5
    lrow = (0.5 + np.random.default_rng(seed).random(n)).astype(np.float32)
    L0 = np.repeat(lrow[:, None], m, axis=1)
    X = T.to_device_X((L0 - np.float32(1)).T, device())
    L = torch.from_numpy(L0).to(device())

    def run(iters):
        fw = T.FrankWolfe(m, n, lam_s, lam_l)
        _, _, t, info = fw.solve(X, L.clone(), 0.0, max_iter=iters, tol=0.0)
        fw.close()
        return t, info

    _, at_start = run(0)  # phi (t = 0) and sigma of the first minimisation
    t, _ = run(1)
    phi, sigma = at_start.F, at_start.sigma
    z = float(lrow.astype(np.float64).sum()) / 16
    gl, l2 = lam_s * m * 16 * z, m * float((lrow.astype(np.float64) ** 2).sum())
    B = phi / lam_l
    dd = B * B * m / sigma ** 2 + 2 * B * m * z / sigma + l2
    eta = (B * sigma + gl - lam_l * B) / dd
    print(f"[fw sums m={m}] eta {t / B:.15g} want {eta:.15g} rel {abs(t / B / eta - 1):.1e}", flush=True)
    assert 0 < eta < 1 and abs(t / B - eta) <= 1e-10 * eta
