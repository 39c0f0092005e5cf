"""The sweep decomposition table (host only): the two splits have entries of their own, a
table saved as rpca_tune_get gives it keeps its meaning, and the no-allocation size limit does
not move with it."""
import ctypes

import pytest

from paper_1702_02241_amd import rpca as R

K_REP = [8, 16, 24, 32]
N_REP = [64, 128, 256, 512, 1024]


@pytest.fixture(autouse=True)
def table():
    saved = {(k, n): (R.rpca_tune_get(k, n)[1:], R.rpca_tune_get_context(k, n)[1:]) for k in K_REP for n in N_REP}
    yield
    for (k, n), (s, c) in saved.items():
        assert R.rpca_tune_set(k, n, *s) == R.RPCA_OK
        assert R.rpca_tune_set_context(k, n, *c) == R.RPCA_OK


@pytest.mark.parametrize("k", K_REP)
@pytest.mark.parametrize("n", N_REP)
def test_default_entries_restore_the_defaults(k, n):
    want = (2048 if k <= 16 else 4096 if n > 512 else 1024, 1)
    assert R.rpca_tune_get(k, n)[1:] == want
    assert R.rpca_tune_get_context(k, n)[1:] == (2048, 1)
    assert R.rpca_tune_set(k, n, *want) == R.RPCA_OK
    assert R.rpca_tune_get_context(k, n)[1:] == (2048, 1)


def test_entries_of_the_two_splits():
    assert R.rpca_tune_set(24, 300, 2048, 2) == R.RPCA_OK
    assert R.rpca_tune_get_context(24, 300)[1:] == (4096, 2)  # twice the default, as the entry
    assert R.rpca_tune_set_context(24, 300, 512, 1) == R.RPCA_OK
    assert R.rpca_tune_get(24, 300)[1:] == (2048, 2)
    assert R.rpca_tune_get_context(20, 511)[1:] == (512, 1)  # same bucket
    assert R.rpca_tune_get_context(24, 600)[1:] == (2048, 1)
    for bad in [(33, 300, 512, 1), (24, 0, 512, 1), (24, 300, 0, 1), (24, 300, (1 << 21) + 1, 1), (24, 300, 512, 17)]:
        assert R.rpca_tune_set_context(*bad) == R.RPCA_EINVAL
    assert R.lib().rpca_tune_get_context(24, 300, None, None) == R.RPCA_EINVAL


@pytest.mark.parametrize("waves,div", [(64, 1), (1 << 20, 16)])
def test_noalloc_limit_does_not_move(waves, div):
    # too large at the default entries (many column chunks), rejected before any device work
    m, n, k = 1 << 20, 1 << 12, 24
    for kk, nn in [(k, n), (16, 200)]:
        assert R.rpca_tune_set(kk, nn, waves, div) == R.RPCA_OK
    dummy = ctypes.c_void_p(16)
    for mm, nn, kk in [(m, n, k), (1 << 23, 300, 16)]:
        assert R.rpca_objgrad_noalloc(mm, nn, kk, 0.1, 1.0, None, dummy, dummy, dummy, dummy, dummy, dummy,
                                      None) == R.RPCA_ETOOBIG
