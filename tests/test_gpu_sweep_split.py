"""GPU parity of the objective/gradient sweep at the edges of its work split.

Each column-group class (chunks of up to 64, 128, 256 and 512 columns), each step class of
the rank (k up to 12, 16, 24, 28, 32) and its edges, waves with no tile, ragged rows and
columns, rows taken in several rounds, and X whose columns are not 16-byte aligned, in both
splits; with a mask, the elastic net and BF16 products.

Bars as in test_gpu_objgrad.py: FP32 1e-5 (sums of at most a few thousand FP32 products of
random sign), BF16 gradients 1e-2 (8-bit significands of G, U and V).
"""
import numpy as np
import pytest
import torch

from oracle import objective as ob
from paper_1702_02241_amd import rpca as R
from paper_1702_02241_amd import synth
from paper_1702_02241_amd import torch_api as T

from gpu_common import device, f32, rel

pytestmark = pytest.mark.gpu

# m, n, k, split: None (the tuning table's), "few" (eight workgroups: rows in rounds) or
# "strips" (an explicit wave count: whole strips to a wave)
SHAPES = [
    (80, 64, 8, None),          # one column group, whole strips
    (333, 65, 12, "few"),       # two groups (3 + 2 tiles), last rank of three steps
    (2050, 130, 13, "few"),     # four groups, m % 4 = 2, first rank of four steps
    (97, 257, 16, None),        # eight groups, seventeen tiles
    (12805, 48, 17, "few"),     # first rank of two blocks, several rounds, m odd
    (640, 513, 24, None),       # two chunks, the second with one column short of its width
    (515, 1025, 25, "few"),     # three chunks
    (1600, 96, 28, "few"),      # rounds of whole strips
    (2101, 512, 29, "few"),     # widest chunk, several rounds
    (1999, 200, 32, "few"),     # largest rank, several rounds
    (200, 35, 25, None),        # three tiles over one group, ragged columns
    (1037, 150, 9, "strips"),   # m odd: columns of every alignment
    (530, 129, 20, "strips"),
]


@pytest.fixture
def split():
    """Context options for a split; the tuning table is put back afterwards."""
    saved = []

    def options(m, n, k, how):
        if how == "few":
            saved.append((k, n) + tuple(R.rpca_tune_get(k, n)[1:]))
            assert R.rpca_tune_set(k, n, 64, 1) == R.RPCA_OK
        return dict(waves=64) if how == "strips" else {}

    yield options
    for k, n, w, d in saved:
        R.rpca_tune_set(k, n, w, d)


def _problem(m, n, k, p_obs=None):
    if p_obs is None:
        p = synth.gaussian_rpca(m=m, n=n, r=min(5, k), k=k, seed=40 + m + n + k)
    else:
        p = synth.partial_rpca(m=m, n=n, r=min(5, k), k=k, p_obs=p_obs, seed=40 + m + n + k)
    return p, synth.random_factors(m, n, k, 5 + k, scale=0.5)


@pytest.mark.parametrize("mode", ["plain", "mask", "elastic", "bf16"])
@pytest.mark.parametrize("m,n,k,how", SHAPES)
def test_objgrad_at_the_edges(m, n, k, how, mode, split):
    p, (U, V) = _problem(m, n, k, 0.4 if mode == "mask" else None)
    mu = 0.3 if mode == "elastic" else 0.0
    dev = device()
    ctx = T.Context(m, n, k, p.lam_s, p.lam_l, p.mask, mu=mu, **split(m, n, k, how))
    # X four bytes past a 16-byte boundary (and, with m % 4 != 0, every column differently)
    buf = torch.empty(m * n + 1, dtype=torch.float32, device=dev)
    Xcm = buf[1:]
    Xcm.copy_(T.to_device_X(p.X, dev).reshape(-1))
    f, gU, gV = ctx.objgrad(Xcm, T.to_device_factor(U, dev), T.to_device_factor(V, dev), R.RPCA_PREC_BF16 if mode == "bf16" else R.RPCA_PREC_FP32)
    torch.cuda.synchronize()
    fr, gUr, gVr = ob.objgrad(f32(U), f32(V), f32(p.X), p.lam_s, p.lam_l, p.mask, mu=mu)
    ef, eu, ev = abs(f.item() - fr) / abs(fr), rel(gU.cpu().numpy(), gUr), rel(gV.cpu().numpy(), gVr)
    print(f"[sweep {mode} {m}x{n} k={k} {how}] f {ef:.2e} gU {eu:.2e} gV {ev:.2e}")
    tol = 1e-2 if mode == "bf16" else 1e-5
    assert ef <= tol and eu <= tol and ev <= tol
    ctx.close()


@pytest.mark.parametrize("m,n,k,how", [(333, 65, 12, "few"), (2050, 130, 13, "few"), (640, 513, 24, None),
                                       (1999, 200, 32, "few"), (1037, 150, 9, "strips")])
@pytest.mark.parametrize("precond", [0, 1])
def test_trial_points_at_the_edges(m, n, k, how, precond, split):
    """A few solver steps: the returned value is the objective at the returned factors (the
    trial sweep forms the point, its gradient's products and its value in one pass), and the
    steps descend."""
    p, (U, V) = _problem(m, n, k)
    dev = device()
    ctx = T.Context(m, n, k, p.lam_s, p.lam_l, **split(m, n, k, how))
    Ud, Vd = T.to_device_factor(U, dev), T.to_device_factor(V, dev)
    rc, info = ctx.solve(T.to_device_X(p.X, dev), Ud, Vd, precond=precond, max_iter=4)
    f0 = ob.objgrad(f32(U), f32(V), f32(p.X), p.lam_s, p.lam_l)[0]
    f1 = ob.objgrad(Ud.cpu().numpy().astype(np.float64), Vd.cpu().numpy().astype(np.float64), f32(p.X), p.lam_s, p.lam_l)[0]
    print(f"[trial {m}x{n} k={k} precond={precond}] rc {rc} f {info.f:.6e} oracle {f1:.6e} start {f0:.6e}")
    assert abs(info.f - f1) <= 1e-5 * abs(f1)
    assert f1 < f0
    ctx.close()
