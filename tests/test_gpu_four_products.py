"""Large FP64 and FP32 contractions (from 8192 x 128 x 16 on, the columns those of the
result's contiguous index) form four real products
for a complex one: the imaginary part carries the rounding of its own terms only.
With three, P3 - P1 - P2, it carries that of the real part, here 10^6 (FP64) and
10^3 (FP32) times its terms.

Bound: a sum of 2 K terms with one rounding each, 2 K u relative to the sum of their
moduli.  Masked launches take narrower tiles with the same products."""
import pytest

pytestmark = pytest.mark.gpu


def _operands(prec, A, B):
    import torch
    td, small = (torch.float64, 1e-6) if prec == "fp64" else (torch.float32, 1e-3)
    g = torch.Generator(device="cuda").manual_seed(sum(A) + 3 * sum(B))
    return [torch.complex(torch.randn(s, generator=g, dtype=td, device="cuda"),
                          small * torch.randn(s, generator=g, dtype=td, device="cuda")) for s in (A, B)]


def _within(prec, C, a, b, K):
    """Whether C's imaginary part is within 2 K u of its terms (a, b: float64 matrices)."""
    import torch
    a, b = a.to(torch.complex128), b.to(torch.complex128)
    want = a.real @ b.imag + a.imag @ b.real
    scale = a.real.abs() @ b.imag.abs() + a.imag.abs() @ b.real.abs()
    u = 2.0 ** (-53 if prec == "fp64" else -24)
    # (the float64 reference has as many roundings)
    return float(((C.imag.double() - want).abs() / scale).max()) < 2 * K * u * (2 if prec == "fp64" else 1)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("M,N,K,Z", [(8192, 128, 16, 1), (8200, 129, 33, 1), (20000, 300, 64, 2), (9001, 128, 65, 1),
                                     (128, 8192, 40, 1), (8192, 128, 700, 1)])
def test_large_products(prec, M, N, K, Z):
    import torch
    import paper_2507_11424_amd as tnb
    A, B = _operands(prec, (Z, M, K), (Z, K, N))
    order = "mn" if M > N else "nm"  # a wide result is the transpose of a tall one
    C = torch.empty((Z, M, N) if M > N else (Z, N, M), dtype=A.dtype, device="cuda")
    h = tnb.Handle(0)
    try:
        h.test_contract(prec, "zmk", A, "zkn", B, "z" + order, C)
        torch.cuda.synchronize()
    finally:
        h.close()
    C = C if M > N else C.mT
    for z in range(Z):
        assert _within(prec, C[z].cpu(), A[z].cpu(), B[z].cpu(), K)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("rows", [144, 160, 192])
def test_masked_large_products(prec, rows):
    import torch
    import paper_2507_11424_amd as tnb
    K = 48
    A, B = _operands(prec, (64, rows, K), (K, 200))
    C = torch.full((64, rows, 200), 5.0, dtype=A.dtype, device="cuda")
    mask = (torch.arange(64, device="cuda") % 3 != 0).to(torch.int32)
    h = tnb.Handle(0)
    try:
        h.test_contract(prec, "zak", A, "kc", B, "zac", C, mask=mask)
        torch.cuda.synchronize()
    finally:
        h.close()
    on = mask.cpu().bool()
    assert _within(prec, C.cpu()[on].reshape(-1, 200), A.cpu()[on].reshape(-1, K), B.cpu(), K)
    assert bool((C.cpu()[~on] == 5.0).all())
