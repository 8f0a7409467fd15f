"""Householder QR in registers for each of its three widths (16, 32 and 64 lanes a row)
and three block heights (32, 64 and 128 rows), on both sides of each edge, and the
levels of its tree below the top: Q^H Q = 1 and Q R = A.

Bounds as for a product of n reflectors of a few roundings each: 64 n u, times sqrt(m)
for Q R relative to the largest entry (complex64 outputs: one rounding of each entry
more, 2^-24 sqrt(m) n at most)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.mark.parametrize("m,n", [(32, 17), (33, 17), (64, 32), (65, 32), (128, 31), (129, 32), (257, 24), (1000, 25),
                                 (5000, 32), (64, 16), (65, 16), (129, 16), (2000, 9), (32, 33), (33, 33), (64, 48),
                                 (65, 50), (17, 30), (16, 40)])
@pytest.mark.parametrize("esz", [16, 8])
def test_widths(m, n, esz):
    import torch
    import paper_2507_11424_amd as tnb
    rng = np.random.default_rng(m * 100 + n)
    A = rng.standard_normal((3, m, n)) + 1j * rng.standard_normal((3, m, n))
    A[1] *= 1e-160 if esz == 16 else 1e-20
    A[2][:, n // 2:] = A[2][:, :n - n // 2]
    td = torch.complex128 if esz == 16 else torch.complex64
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
    tol = 64 * n * U + (2.0 ** -24 * np.sqrt(m) * n if esz == 8 else 0.0)
    for b in range(3):
        s = np.abs(a[b]).max()
        assert np.abs(q[b].conj().T @ q[b] - np.eye(k)).max() < tol, b
        assert np.abs(q[b] @ (r[b] / s) - a[b] / s).max() < tol * np.sqrt(m), b
        assert np.abs(np.tril(r[b], -1)).max() == 0.0
