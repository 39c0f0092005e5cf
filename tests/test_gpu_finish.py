"""GPU parity of the finishing reduction at the edges of its block split.

Workgroup rows from one to more than the sixteen slices of sixteen that a block sums at
once; ranks whose rows of V do not fill a wave; several column chunks.  Bars as in
test_gpu_objgrad.py (the sums run in 64 bits, so the sweep's FP32 products decide: 1e-5).
Repeated calls return the same bits: the arrival counter is back at zero.
"""
import pytest
import torch

from oracle import objective as ob
from paper_1702_02241_amd import synth
from paper_1702_02241_amd import torch_api as T

from gpu_common import device, f32, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,waves", [
    (40, 33, 1, 4),        # one workgroup row, 64 rows of V a wave
    (300, 70, 7, 64),      # sixteen rows: one slice, sixteen groups
    (1100, 70, 7, 68),     # seventeen rows: two slices, the second nearly empty
    (16500, 20, 5, 1024),  # 256 rows: sixteen slices
    (17000, 20, 5, 1060),  # 265 rows: a second pass
    (70000, 40, 3, 4200),  # 1,050 rows: several passes
    (900, 300, 22, 512),   # two rows of V a wave, several chunks
    (600, 130, 32, 256),   # two rows of V fill the wave
])
def test_reduction_matches_oracle_and_repeats(m, n, k, waves):
    p = synth.gaussian_rpca(m=m, n=n, r=min(3, k), k=k, seed=70 + m + n)
    U, V = synth.random_factors(m, n, k, 3 + k, scale=0.5)
    dev = device()
    ctx = T.Context(m, n, k, p.lam_s, p.lam_l, waves=waves)
    Xcm, Ud, Vd = T.to_device_X(p.X, dev), T.to_device_factor(U, dev), T.to_device_factor(V, dev)
    f, gU, gV = ctx.objgrad(Xcm, Ud, Vd)
    f2, gU2, gV2 = ctx.objgrad(Xcm, Ud, Vd)
    torch.cuda.synchronize()
    fr, gUr, gVr = ob.objgrad(f32(U), f32(V), f32(p.X), p.lam_s, p.lam_l)
    ef, eu, ev = abs(f.item() - fr) / abs(fr), rel(gU.cpu().numpy(), gUr), rel(gV.cpu().numpy(), gVr)
    print(f"[finish {m}x{n} k={k} waves={waves}] f {ef:.2e} gU {eu:.2e} gV {ev:.2e}")
    assert ef <= 1e-5 and eu <= 1e-5 and ev <= 1e-5
    assert torch.equal(f, f2) and torch.equal(gU, gU2) and torch.equal(gV, gV2)
    ctx.close()
