"""Orthonormalisation and factorisation in little memory: whatever allocation fails,
all workspace is given back, so that the factorisation's second way (Householder,
which needs less) and the next call start from all of it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method,m,n", [("factor", 600, 40), ("cholesky", 600, 40), ("cholesky", 200, 20)])
def test_capped(method, m, n):
    import torch
    import paper_2507_11424_amd as tnb
    rng = np.random.default_rng(m + n)
    A = torch.from_numpy(rng.standard_normal((2, m, n)) + 1j * rng.standard_normal((2, m, n))).cuda()
    Q = torch.empty_like(A)
    R = torch.empty((2, n, n), dtype=A.dtype, device="cuda") if method == "factor" else None
    failed = worked = 0
    for kib in [1, 2] + list(range(64, 6144, 64)):
        h = tnb.Handle(0)
        try:
            h.test_workspace(kib << 10)
            try:
                h.test_qr(A, Q, R, method=method)
                worked += 1
                torch.cuda.synchronize()
                assert float((Q.mH @ Q - torch.eye(n, device="cuda")).abs().max()) < 1e-12
                if R is not None:
                    assert float((Q @ R - A).abs().max()) < 1e-11
            except tnb.TnError as e:
                assert e.status == 3
                failed += 1
            assert h.test_workspace(0) == 0, kib
        finally:
            h.close()
    assert failed and worked
