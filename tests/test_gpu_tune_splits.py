"""GPU test of the tuning table's two splits: batches read the entries for whole strips a wave
(wave count over 1024 as a factor), other contexts the entries of the split by columns, ranks
above 16 and several chunks among them; the autotuner leaves every entry of both at one of its
candidates; an evaluation without allocation is accepted whatever the table holds.
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

K_REP = [8, 16, 24, 32]
N_REP = [64, 128, 256, 512, 1024]


@pytest.fixture(autouse=True)
def table():
    device()
    saved = {(k, n): (R.rpca_tune_get(k, n)[1:], R.rpca_tune_get_context(k, n)[1:]) for k in K_REP for n in N_REP}
    yield
    for (k, n), (s, c) in saved.items():
        assert R.rpca_tune_set(k, n, *s) == R.RPCA_OK
        assert R.rpca_tune_set_context(k, n, *c) == R.RPCA_OK


def _batch_waves(m, n, k):
    B = T.Batch([(m, n, k)], [0.05], [1.0])
    w = B.instance_waves(0)
    B.close()
    return w


def _layout(m, n, k, waves=None):
    c = T.Context(m, n, k, 0.05, 1.0, waves=waves)
    rc, lay = R.rpca_sweep_layout(c.ctx)
    c.close()
    assert rc == R.RPCA_OK
    return lay


@pytest.mark.parametrize("m,n,k,default", [(8192, 300, 24, 1024), (8192, 1024, 24, 4096), (8192, 200, 10, 2048)])
def test_batches_and_contexts_read_their_own_entries(m, n, k, default):
    waves, lay, strips = _batch_waves(m, n, k), _layout(m, n, k), _layout(m, n, k, waves=512)
    # a table saved with the default entry changes nothing
    assert R.rpca_tune_set(k, n, default, 1) == R.RPCA_OK
    assert (_batch_waves(m, n, k), _layout(m, n, k)) == (waves, lay)
    # the share: entry / 1024 times the chip's waves, at least four strips a wave
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for entry in (512, 1024, 2048, 4096):
        assert R.rpca_tune_set(k, n, entry, 1) == R.RPCA_OK
        assert _batch_waves(m, n, k) == min(round(16 * cus * entry / 1024), int(entry / 1024 * (m // 16)) // 4)
    # the context entry moves contexts alone
    assert R.rpca_tune_set(k, n, default, 1) == R.RPCA_OK
    assert R.rpca_tune_set_context(k, n, 512, 2) == R.RPCA_OK
    assert _batch_waves(m, n, k) == waves and _layout(m, n, k, waves=512) == strips
    got = _layout(m, n, k)
    assert got[0] * got[3] < lay[0] * lay[3] and got[2] < lay[2]


def test_autotune_leaves_both_splits_at_candidates():
    rc = R.rpca_autotune(2048, 1, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == R.RPCA_OK
    for k in K_REP:
        for n in N_REP:
            for get in (R.rpca_tune_get, R.rpca_tune_get_context):
                _, w, d = get(k, n)
                assert w in (1024, 2048, 4096) and d in (1, 2)


def test_noalloc_is_accepted_whatever_the_table_holds():
    # the context entry's partials (one workgroup row a strip) would not fit the array
    p = synth.gaussian_rpca(m=40000, n=400, r=5, k=25, seed=9)
    assert R.rpca_tune_set_context(p.k, p.n, 1 << 21, 16) == R.RPCA_OK
    U, V = synth.random_factors(p.m, p.n, p.k, 3, scale=0.4)
    dev = device()
    X, Ud, Vd = T.to_device_X(p.X, dev), T.to_device_factor(U, dev), T.to_device_factor(V, dev)
    f = torch.zeros(1, dtype=torch.float64, device=dev)
    gU, gV = torch.empty_like(Ud), torch.empty_like(Vd)
    rc = R.rpca_objgrad_noalloc(p.m, p.n, p.k, p.lam_s, p.lam_l, None, X.data_ptr(), Ud.data_ptr(), Vd.data_ptr(),
                                f.data_ptr(), gU.data_ptr(), gV.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert rc == R.RPCA_OK
    torch.cuda.synchronize()
    fr, gUr, gVr = ob.objgrad(f32(U), f32(V), f32(p.X), p.lam_s, p.lam_l)
    assert abs(f.item() - fr) <= 1e-5 * abs(fr)
    assert rel(gU.cpu().numpy(), gUr) <= 1e-5 and rel(gV.cpu().numpy(), gVr) <= 1e-5
