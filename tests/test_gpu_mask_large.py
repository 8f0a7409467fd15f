"""A masked contraction of narrow items near the largest that one launch takes (2^31
entries of the result): more 16x16 tiles than a launch has threads for, so every
item is computed."""
import pytest

pytestmark = pytest.mark.gpu


def test_narrow_items_of_a_huge_result():
    import torch
    import paper_2507_11424_amd as tnb
    Z, rows, K, N = 1 << 17, 16, 100, 1023
    g = torch.Generator(device="cuda").manual_seed(1)
    A = torch.randn((Z, rows, K), generator=g, dtype=torch.complex64, device="cuda")
    B = torch.randn((K, N), generator=g, dtype=torch.complex64, device="cuda")
    C = torch.empty((Z, rows, N), dtype=torch.complex64, device="cuda")
    mask = (torch.arange(Z, device="cuda") % 3 != 0).to(torch.int32)
    h = tnb.Handle(0)
    try:
        h.test_contract("fp32", "zak", A, "kc", B, "zac", C, mask=mask)
        torch.cuda.synchronize()
    finally:
        h.close()
    some = torch.tensor([1, 2, 4, 1000, 65536, 131069, 131071], device="cuda")
    assert bool(mask[some].all())
    a, b = A[some].to(torch.complex128).cpu(), B.to(torch.complex128).cpu()
    err = (C[some].to(torch.complex128).cpu() - a @ b).abs() / (a.abs() @ b.abs())
    assert float(err.max()) < 4 * K * 2.0 ** -24
