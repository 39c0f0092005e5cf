"""Infinite entries in the objective/gradient: f and every entry of the gradients are finite,
infinite or NaN exactly where the same sums in 64 bits are.

An infinite U_iq makes row i of U V^T infinite, so f is infinite and G's row i is at the
threshold: only column q of the gradients becomes infinite.  A solver's line search tells an
overflowing step (f infinite) from a failed evaluation (f not a number).  The shapes give a
workgroup more column groups than some chunk has tiles, so that waves without a tile meet the
infinity too.  Finite entries: the FP32 bar of test_gpu_objgrad.py (1e-5; BF16 products 1e-2).
"""
import numpy as np
import pytest
import torch

from oracle import objective as ob
from paper_1702_02241_amd import rpca as R
from paper_1702_02241_amd import synth
from paper_1702_02241_amd import torch_api as T

from gpu_common import device, f32

pytestmark = pytest.mark.gpu


def _kinds(a):
    a = np.asarray(a, np.float64)
    return np.where(np.isnan(a), 2, np.where(np.isinf(a), np.sign(a), 0))


def _want(U, V, X, lam_s, lam_l, mu):
    """f and the gradients in 64 bits (the oracle's sums; its Huber value multiplies the
    distance past the threshold by a zero slope, which has no value at infinity)."""
    U, V, X = f32(U), f32(V), f32(X)
    with np.errstate(invalid="ignore"):
        Rs = U @ V.T - X
        c = np.clip(Rs, -lam_s, lam_s)
        rho = c * (Rs - 0.5 * c)
        if mu:
            rho = rho + 0.5 * ob.kappa_of(mu) * (Rs - c) ** 2
        G = ob.huber_deriv(Rs, lam_s, mu)
        f = rho.sum() + 0.5 * lam_l * (np.sum(U * U) + np.sum(V * V))
        return f, G @ V + lam_l * U, G.T @ U + lam_l * V


def _check(got, want, tol, what):
    got, want = np.asarray(got, np.float64), np.asarray(want, np.float64)
    assert np.array_equal(_kinds(got), _kinds(want)), what
    fin = np.isfinite(want)
    if fin.any():
        assert np.linalg.norm(got[fin] - want[fin]) <= tol * np.linalg.norm(want[fin]), what


SHAPES = [(48, 80, 5), (96, 112, 10), (64, 80, 13), (128, 80, 26), (304, 144, 20)]


# (BF16 up to rank 16 splits U and V into two bf16 parts, which an infinity does not have)
@pytest.mark.parametrize("m,n,k,mode", [s + (mode,) for s in SHAPES for mode in ("plain", "elastic")]
                         + [s + ("bf16",) for s in SHAPES if s[2] > 16])
@pytest.mark.parametrize("where", ["U", "V"])
def test_infinite_factor_entry(m, n, k, mode, where):
    p = synth.gaussian_rpca(m=m, n=n, r=min(5, k), k=k, seed=m + k)
    U, V = synth.random_factors(m, n, k, 3 + k, scale=0.5)
    if where == "U":
        U[m // 3, k // 2] = np.inf
    else:
        V[1, k // 2] = np.inf  # a column of the first tile
    mu = 0.3 if mode == "elastic" else 0.0
    dev = device()
    ctx = T.Context(m, n, k, p.lam_s, p.lam_l, mu=mu)
    f, gU, gV = ctx.objgrad(T.to_device_X(p.X, dev), T.to_device_factor(U, dev), T.to_device_factor(V, dev),
                            R.RPCA_PREC_BF16 if mode == "bf16" else R.RPCA_PREC_FP32)
    torch.cuda.synchronize()
    fr, gUr, gVr = _want(U, V, p.X, p.lam_s, p.lam_l, mu)
    assert fr == np.inf
    print(f"[nonfinite {mode} {m}x{n} k={k} {where}] f {f.item()}", flush=True)
    tol = 1e-2 if mode == "bf16" else 1e-5
    _check(f.item(), fr, tol, "f")
    _check(gU.cpu().numpy(), gUr, tol, "gU")
    _check(gV.cpu().numpy(), gVr, tol, "gV")
    ctx.close()


@pytest.mark.parametrize("mode", ["plain", "bf16"])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("val", [np.inf, -np.inf, 3e38])
@pytest.mark.parametrize("m,n,k", [(128, 80, 26), (300, 144, 20), (512, 528, 25), (256, 200, 10)])
def test_objective_past_overflow(m, n, k, val, masked, mode):
    """One huge entry of X and a threshold of 1e20: the entry's value, 1e20 |X|, is past FP32."""
    p = synth.gaussian_rpca(m=m, n=n, r=5, k=k, seed=m + k)
    U, V = synth.random_factors(m, n, k, 3 + k, scale=0.5)
    X = np.array(p.X)
    X[m // 3, n // 2] = val
    mask = None
    if masked:
        mask = (np.random.default_rng(k).random((m, n)) < 0.7).astype(np.uint8)
        mask[m // 3, n // 2] = 1
    dev = device()
    ctx = T.Context(m, n, k, 1e20, p.lam_l, mask)
    f, _, _ = ctx.objgrad(T.to_device_X(X, dev), T.to_device_factor(U, dev), T.to_device_factor(V, dev),
                          R.RPCA_PREC_BF16 if mode == "bf16" else R.RPCA_PREC_FP32)
    torch.cuda.synchronize()
    print(f"[overflow {m}x{n} k={k} {val}] f {f.item()}", flush=True)
    assert f.item() == np.inf
    ctx.close()
