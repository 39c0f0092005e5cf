"""GPU parity of the fused G^T G pass at the edges of its work split.

Column groups of one, two and four waves (n up to 64, 128, 256), ragged last tiles, odd row
counts (columns of every alignment), fewer strips than row lanes; the data source through
Frank-Wolfe's linear minimisation, the residual source (k up to 12, 13 and 16, masked,
elastic net) through the certificate's power iteration.

Bars as in test_gpu_fw.py and test_gpu_solve.py: sigma of the start to 1e-5; the leading Ritz
value a lower bound of the top singular value (to rounding) and within 1e-3 of it, 1e-2 where
that value is below 0.9 and the iteration may stop early; T4 to 1e-3 where the largest block
of 32 vectors holds every singular value above one.
"""
import numpy as np
import pytest


from oracle import certificate as ce
from oracle import frank_wolfe as fw
from oracle import lbfgs as lb
from oracle import objective as ob
from oracle import rsvd as rs
from paper_1702_02241_amd import rpca as R
from paper_1702_02241_amd import synth
from paper_1702_02241_amd import torch_api as T

from gpu_common import device, f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,masked", [(16, 16, False), (40, 33, True), (131, 64, False), (1001, 65, False),
                                        (257, 128, True), (2003, 129, False), (4161, 256, True)])
def test_data_source(m, n, masked):
    p = (synth.partial_rpca(m=m, n=n, r=4, k=4, p_obs=0.75, seed=m + n) if masked else
         synth.gaussian_rpca(m=m, n=n, r=4, k=4, seed=m + n, lam_s=0.3, lam_l=1.5))
    X = f32(p.X)
    solver = T.FrankWolfe(p.m, p.n, p.lam_s, p.lam_l, mask=p.mask)
    Xcm = T.to_device_X(p.X, device())
    rc, _, _, info = solver.solve(Xcm, max_iter=0, tol=0.0, power_tol=3e-6)
    _, _, o = fw.fw_iteration(np.zeros((m, n)), 0.0, X, p.lam_s, p.lam_l, p.mask)
    print(f"[gram data {m}x{n} mask={masked}] sigma {info.sigma:.9g} oracle {o['sigma']:.9g} power {info.power_iters}")
    assert rc == R.RPCA_ENOTCONV
    assert abs(info.sigma - o["sigma"]) <= 1e-5 * o["sigma"]
    solver.close()


@pytest.mark.parametrize("m,n,k,p_obs,mu", [
    (90, 40, 4, None, 0.0), (401, 65, 12, None, 0.0), (1203, 128, 13, 0.8, 0.0), (533, 129, 16, None, 0.3),
    (2050, 256, 9, 0.7, 0.2),
])
def test_residual_source(m, n, k, p_obs, mu):
    if p_obs is None:
        p = synth.gaussian_rpca(m=m, n=n, r=max(1, k - 3), k=k, seed=50 + m, lam_s=1.0 / np.sqrt(max(m, n)))
    else:
        p = synth.partial_rpca(m=m, n=n, r=max(1, k - 3), k=k, p_obs=p_obs, seed=50 + m)
    U0, V0 = rs.rsvd_factors(p.X, k, synth.gaussian_matrix(n, k + 5, 12), mask=p.mask)
    res = lb.lbfgs(lambda x: _fg(x, p, mu), ob.pack(U0, V0), max_iter=25)
    U, V = ob.unpack(res["x"], m, n, k)
    dev = device()
    ctx = T.Context(m, n, k, p.lam_s, p.lam_l, mask=p.mask, mu=mu)
    c = ctx.certificate(T.to_device_X(p.X, dev), T.to_device_factor(U, dev), T.to_device_factor(V, dev))
    o = ce.certificate(f32(U), f32(V), f32(p.X), p.lam_s, p.lam_l, mask=p.mask, tau=1e-6, mu=mu)
    sv0 = o["sv_perp"][0]
    print(f"[gram resid {m}x{n} k={k} p_obs={p_obs} mu={mu}] theta0 {c.theta[0]:.8g} sv0 {sv0:.8g} "
          f"T4 {c.T4:.6g} oracle {o['T4']:.6g} steps {c.power_iters}")
    assert c.theta[0] <= sv0 * (1 + 1e-6) + 1e-9
    assert abs(c.theta[0] - sv0) <= (1e-2 if sv0 < 0.9 else 1e-3) * sv0 + 1e-5
    if (o["sv_perp"] > 1).sum() < 32:
        assert abs(c.T4 - o["T4"]) <= 1e-3 * max(o["T4"], 1.0) + 1e-9
    else:  # more singular values above one than the largest block holds: T4 is an upper bound
        assert c.T4 >= o["T4"]
    ctx.close()


def _fg(x, p, mu):
    U, V = ob.unpack(x, p.m, p.n, p.k)
    f, gU, gV = ob.objgrad(U, V, p.X, p.lam_s, p.lam_l, p.mask, mu=mu)
    return f, ob.pack(gU, gV)
