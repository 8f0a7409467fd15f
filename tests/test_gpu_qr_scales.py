"""Householder QR in registers on columns so small that squares underflow: pivots
whose square is subnormal beside a column whose sum of squares is not, columns far
smaller than the ones before them, subnormal entries.

Bounds: a reflector is unitary to a few roundings and Q is a product of n of them on
up to 128 rows, 64 n u for Q^H Q - 1; columns agree with Q R to the same times
sqrt(m), each relative to its own norm."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _factor(A):
    import torch
    import paper_2507_11424_amd as tnb
    dA = torch.from_numpy(A).cuda()
    z, m, n = A.shape
    k = min(m, n)
    Q = torch.empty((z, m, k), dtype=dA.dtype, device="cuda")
    R = torch.empty((z, k, n), dtype=dA.dtype, device="cuda")
    h = tnb.Handle(0)
    try:
        h.test_qr(dA, Q, R, method="householder")
        torch.cuda.synchronize()
    finally:
        h.close()
    return Q.cpu().numpy(), R.cpu().numpy()


def _check(A, q, r):
    m, n = A.shape[1:]
    k = min(m, n)
    for b in range(A.shape[0]):
        assert np.abs(q[b].conj().T @ q[b] - np.eye(k)).max() < 64 * n * U, b
        s = np.abs(A[b]).max(axis=0)  # per column
        s = np.where(s > 0, s, 1.0)
        assert np.abs(q[b] @ (r[b] / s) - A[b] / s).max() < 64 * n * U * np.sqrt(m), b


@pytest.mark.parametrize("m,n", [(64, 1), (20, 2), (100, 16), (128, 33)])
def test_subnormal_pivot_square(m, n):
    rng = np.random.default_rng(m + n)
    A = rng.standard_normal((40, m, n)) + 1j * rng.standard_normal((40, m, n))
    # column 0: norm just above 1e-140, its pivot 1.2e-156 .. 2e-156 at any phase
    A[:, 0, 0] = 0.0
    A[:, :, 0] *= (1.005e-140 / np.linalg.norm(A[:, :, 0], axis=1))[:, None]
    A[:, 0, 0] = rng.uniform(1.2, 2.0, 40) * 1e-156 * np.exp(2j * np.pi * rng.uniform(size=40))
    A[:, :, 1:] *= 1e-140
    _check(A, *_factor(A))


@pytest.mark.parametrize("m,n", [(16, 3), (64, 16), (129, 20), (128, 64)])
@pytest.mark.parametrize("span", [(-140, -40), (-95, -105), (-200, 100), (-150, -290), (140, -290)])
def test_graded_columns(m, n, span):
    rng = np.random.default_rng(m + n)
    A = rng.standard_normal((3, m, n)) + 1j * rng.standard_normal((3, m, n))
    A = A * np.logspace(*span, n)
    _check(A, *_factor(A))
