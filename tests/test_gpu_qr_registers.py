"""Householder QR with its blocks in registers, at the edges of its two block
heights (32 and 128 rows), of the tree's levels and of the 64 columns, in both
layouts of the fit (QR and, through conjugate-transposed strides, LQ), against
the factorisation's own properties: Q^H Q = 1 and Q R = A."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(1, 1), (4, 4), (5, 9), (31, 16), (32, 32), (33, 16), (64, 64), (65, 1), (127, 63),
                                 (128, 64), (129, 64), (257, 64), (300, 50), (1000, 3), (5000, 64)])
@pytest.mark.parametrize("esz", [16, 8])
def test_qr_registers(m, n, esz):
    import torch
    import paper_2507_11424_amd as tnb
    rng = np.random.default_rng(m * 100 + n)
    A = rng.standard_normal((3, m, n)) + 1j * rng.standard_normal((3, m, n))
    A[1] *= 1e-160                               # squares underflow: the scaled step
    A[2][:, n // 2:] = A[2][:, :n - n // 2]      # rank deficient
    if n > 1:
        A[2][:, 0] = 0.0                         # a zero column
    td = torch.complex128 if esz == 16 else torch.complex64
    if esz == 8:
        A[1] *= 1e140
    dA = torch.from_numpy(A).to(td).cuda()
    k = min(m, n)
    Q = torch.empty((3, m, k), dtype=td, device="cuda")
    R = torch.empty((3, k, n), dtype=td, device="cuda")
    h = tnb.Handle(0)
    try:
        h.test_qr(dA, Q, R, method="householder")
        torch.cuda.synchronize()
    finally:
        h.close()
    a, q, r = (x.cpu().numpy().astype(np.complex128) for x in (dA, Q, R))
    # FP64 arithmetic: a few n u per column; complex64 outputs are rounded once
    tol = 1e-13 * max(n, 8) if esz == 16 else 3e-6
    for b in range(3):
        s = np.abs(a[b]).max()
        assert np.abs(q[b].conj().T @ q[b] - np.eye(k)).max() < tol, b
        assert np.abs(q[b] @ (r[b] / s) - a[b] / s).max() < tol * np.sqrt(m), b
        assert np.abs(np.tril(r[b], -1)).max() == 0.0
