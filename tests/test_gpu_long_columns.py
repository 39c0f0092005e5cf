"""GPU parity of the objective/gradient sweep and of the fused Gram pass (certificate) on columns
of 2^24 rows and more, where a wave's columns together pass 32-bit byte offsets unless it has
few of them, and of 2^26 rows, where one tile of columns does and X is read by address.

The reference is the same sums in 64 bits on the device, in row chunks.  Bar: 1e-5 (FP32 sums
of at most 4096 strips a row lane, of random sign: 64 roundings of 6e-8 at each stage).
"""
import pytest
import torch

from paper_1702_02241_amd import rpca as R
from paper_1702_02241_amd import torch_api as T

from gpu_common import device

pytestmark = pytest.mark.gpu

CHUNK = 1 << 22


def _data(m, n, k, masked, seed):
    dev = device()
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    U = 0.5 * torch.randn(m, k, generator=g, device=dev)
    V = 0.5 * torch.randn(n, k, generator=g, device=dev)
    X = torch.empty(n, m, device=dev)
    for j in range(n):
        X[j] = torch.randn(m, generator=g, device=dev)
    bits = on = None
    if masked:
        mw = (m + 31) // 32
        bits = torch.randint(-2**31, 2**31 - 1, (n, mw), dtype=torch.int32, generator=g, device=dev)
    return X, U, V, bits


def _observed(bits, r0, r1):
    """Rows r0 (a multiple of 32) .. r1 of the mask as 0/1 doubles, (n, r1 - r0)."""
    w = bits[:, r0 // 32:(r1 + 31) // 32]
    b = (w[:, :, None] >> torch.arange(32, dtype=torch.int32, device=w.device)) & 1
    return b.reshape(w.shape[0], -1)[:, :r1 - r0].double()


def _residual_chunks(X, U, V, bits, lam_s):
    for r0 in range(0, X.shape[1], CHUNK):
        r1 = min(X.shape[1], r0 + CHUNK)
        Rs = V.double() @ U[r0:r1].double().T - X[:, r0:r1].double()
        on = _observed(bits, r0, r1) if bits is not None else 1.0
        c = Rs.clamp(-lam_s, lam_s)
        yield r0, r1, (c * (Rs - 0.5 * c) * on), c * on


def _rel(a, b):
    return float((a.double() - b).norm() / b.norm())


@pytest.mark.parametrize("m,n,k,masked", [
    ((1 << 24) + 5, 17, 2, False),   # two tiles: one wave past the limit of four
    ((1 << 24) + 5, 17, 2, True),
    ((1 << 24) + 48, 70, 3, False),  # five tiles, two to a wave
    ((1 << 25) + 7, 16, 13, False),  # one tile
    ((1 << 25) + 7, 33, 18, True),   # three tiles to a wave, two blocks of ranks: by address, whole and ragged strips
    ((1 << 26) + 21, 2, 2, True),    # one tile by address
])
def test_objgrad(m, n, k, masked):
    X, U, V, bits = _data(m, n, k, masked, m % 1000 + n)
    lam_s, lam_l = 0.7, 1.0
    ctx = T.Context(m, n, k, lam_s, lam_l, mask_bits=bits)
    f, gU, gV = ctx.objgrad(X, U, V)
    torch.cuda.synchronize()
    ctx.close()
    fr, eu, nu = 0.5 * lam_l * float(U.double().square().sum() + V.double().square().sum()), 0.0, 0.0
    gVr = lam_l * V.double()
    for r0, r1, rho, G in _residual_chunks(X, U, V, bits, lam_s):
        fr += float(rho.sum())
        ref = G.T @ V.double() + lam_l * U[r0:r1].double()
        eu += float((gU[r0:r1].double() - ref).square().sum())
        nu += float(ref.square().sum())
        gVr += G @ U[r0:r1].double()
    ef, eu, ev = abs(f.item() - fr) / fr, (eu / nu) ** 0.5, _rel(gV, gVr)
    print(f"[long columns {m}x{n} k={k} mask={masked}] f {ef:.1e} gU {eu:.1e} gV {ev:.1e}", flush=True)
    assert ef <= 1e-5 and eu <= 1e-5 and ev <= 1e-5


@pytest.mark.parametrize("m,n,k,masked", [((1 << 24) + 5, 17, 2, False), ((1 << 24) + 5, 16, 2, True),
                                          ((1 << 26) + 21, 3, 1, False)])
def test_certificate_gram_pass(m, n, k, masked):
    X, U, V, bits = _data(m, n, k, masked, m % 1000 + n)
    lam_s = 0.7
    # singular values of lam_l M = P_perp(G) from (I - V1 V1^T)(G^T G - B^T B)(I - V1 V1^T), B = U1^T G
    U1, V1 = torch.linalg.qr(U.double())[0], torch.linalg.qr(V.double())[0]
    W, B = torch.zeros(n, n, dtype=torch.float64, device=U.device), torch.zeros(k, n, dtype=torch.float64, device=U.device)
    for r0, r1, _, G in _residual_chunks(X, U, V, bits, lam_s):
        W += G @ G.T
        B += U1[r0:r1].T @ G.T
    P = torch.eye(n, dtype=torch.float64, device=U.device) - V1 @ V1.T
    s = torch.linalg.eigvalsh(P @ (W - B.T @ B) @ P).clamp_min(0).sqrt()
    lam_l = 0.5 * float(s[-1])  # singular values of M up to 2: T4 is not zero
    want = float((s / lam_l - 1).clamp_min(0).square().sum())
    ctx = T.Context(m, n, k, lam_s, lam_l, mask_bits=bits)
    c = ctx.certificate(X, U, V)
    ctx.close()
    print(f"[long columns, T4 {m}x{n} k={k} mask={masked}] {c.T4:.8g} {want:.8g}", flush=True)
    # the certificate tests' bar
    assert want > 0.5 and abs(c.T4 - want) <= 1e-3 * max(want, 1.0)
