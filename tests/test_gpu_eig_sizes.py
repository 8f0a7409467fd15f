"""The loop-error eigenvalue kernel where its variants meet: one wave up to 64
columns, four waves with the matrix in LDS up to 96, in global memory above;
and matrices far from unit scale."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 63, 65, 81, 96, 97, 225])
@pytest.mark.parametrize("scale", [1.0, 1e-180, 1e150])
def test_eig_kernel_variants(n, scale):
    import torch
    import paper_2507_11424_amd as tnb
    rng = np.random.default_rng(n)
    A = rng.standard_normal((3, n, n)) + 1j * rng.standard_normal((3, n, n))
    A[1] = A[1] @ A[1].conj().T               # Hermitian positive: real eigenvalues
    A[2, :, : n // 2] = 0.0                   # rank n - n / 2: a block of zero eigenvalues
    h = tnb.Handle(0)
    try:
        lam, eps, info = (x.cpu().numpy() for x in h.test_eig(torch.from_numpy(A * scale).cuda()))
    finally:
        h.close()
    assert np.all(info == 0)
    for q in range(3):
        ref = np.linalg.eigvals(A[q])
        a = np.sort(np.abs(ref))
        got = np.sort(np.abs(lam[q] / scale))
        # backward stable: every modulus within a small multiple of n u ||A||, the
        # defective zeros of the last matrix excluded
        k = n // 2 if q == 2 else 0
        assert np.abs(got[k:] - a[k:]).max() < 1e-10 * np.linalg.norm(A[q], 2), q
        assert abs(eps[q] - (1 - a[-1] / a.sum())) < 1e-10
