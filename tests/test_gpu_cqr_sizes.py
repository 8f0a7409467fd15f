"""CholeskyQR at the edges of its block counts (16 columns a block), of the rows a
workgroup stages (32) and of the one-launch form (32 columns, 256 rows), in both
layouts of the fit, with well and ill conditioned items and a rank-deficient one
(refactored by Householder) in one batch: Q^H Q = 1 and the span of Q holds A."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(1, 1), (16, 16), (17, 16), (40, 17), (255, 32), (256, 32), (257, 32), (256, 33),
                                 (48, 48), (100, 49), (64, 64), (65, 64), (1025, 64), (2048, 27)])
@pytest.mark.parametrize("method", ["cholesky", "cholesky_lq"])
@pytest.mark.parametrize("esz", [16, 8])
def test_cqr_sizes(m, n, method, esz):
    import torch
    import paper_2507_11424_amd as tnb
    rng = np.random.default_rng(100 * m + n)
    A = rng.standard_normal((3, m, n)) + 1j * rng.standard_normal((3, m, n))
    if n > 1:
        u, _ = np.linalg.qr(A[1])
        v, _ = np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))
        A[1] = (u * np.logspace(0, -8, n)) @ v
        A[2][:, n // 2:] = A[2][:, :n - n // 2]
    A[1] *= 1e-30
    td = torch.complex128 if esz == 16 else torch.complex64
    lq = method == "cholesky_lq"
    host = torch.from_numpy(A).to(td)
    dA = (host.mH if lq else host).contiguous().cuda()
    Q = torch.empty_like(dA)
    h = tnb.Handle(0)
    try:
        h.test_qr(dA, Q, None, method=method)
        torch.cuda.synchronize()
    finally:
        h.close()
    q = Q.cpu().numpy().astype(np.complex128)
    if lq:
        q = q.conj().swapaxes(1, 2)
    a = host.numpy().astype(np.complex128)
    tol = 1e-12 if esz == 16 else 1e-5
    for b in range(3):
        assert np.abs(q[b].conj().T @ q[b] - np.eye(n)).max() < tol * 10, b
        s = np.abs(a[b]).max()
        assert np.abs(q[b] @ (q[b].conj().T @ a[b]) - a[b]).max() < tol * 10 * s, b
