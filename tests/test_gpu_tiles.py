"""The 32x32 and 64x128 tiles of the contraction kernel, and the planner's own
choice on both sides of each line of its rule, against a float64 product; masked
launches whose items are narrower than the planned tile."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# relative to sum |a||b|, as for the other tiles
TOL = {"fp64": 1e-12, "fp32": 3e-6, "bf16x3": 3e-5, "bf16x6": 3e-6}


@pytest.fixture(scope="module")
def handle():
    import paper_2507_11424_amd as tnb
    h = tnb.Handle(0)
    yield h
    h.close()


def _run(handle, prec, M, N, K, Z, order="mn", **kw):
    import torch
    td = torch.complex128 if prec == "fp64" else torch.complex64
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    A = torch.randn((Z, M, K), generator=g, dtype=td, device="cuda")
    B = torch.randn((Z, K, N), generator=g, dtype=td, device="cuda")
    C = torch.full((Z, M, N) if order == "mn" else (Z, N, M), 5.0, dtype=td, device="cuda")
    handle.test_contract(prec, "zmk", A, "zkn", B, "z" + order, C, conjA=True, **kw)
    got = C if order == "mn" else C.mT
    a, b = A.to(torch.complex128).cpu(), B.to(torch.complex128).cpu()
    err = (got.to(torch.complex128).cpu() - torch.bmm(a.conj().resolve_conj(), b)).abs()
    scale = torch.bmm(a.abs(), b.abs())
    assert float((err / scale).max()) < TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("M,N,K,Z", [(1, 1, 5, 1), (33, 65, 70, 2), (130, 200, 97, 1), (31, 129, 4100, 1)])
@pytest.mark.parametrize("cfg", [5, 6, 8])
@pytest.mark.parametrize("ksplit", [1, 3])
def test_new_tiles(handle, prec, M, N, K, Z, cfg, ksplit):
    if cfg == 6 and not prec.startswith("bf16"):
        pytest.skip("the 64x128 tile exists for split-BF16 only")
    if cfg == 8 and prec.startswith("bf16"):
        pytest.skip("the 64x32 tile exists for FP64 and FP32 only")
    _run(handle, prec, M, N, K, Z, cfg=cfg, ksplit=ksplit)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("M,N,K,Z", [
    (64, 16, 300, 1), (64, 17, 191, 1), (64, 17, 192, 1), (700, 40, 64, 1), (63, 40, 64, 1), (700, 40, 65, 1),
    (16384, 32, 33, 1), (16384, 33, 32, 1), (32, 16384, 40, 1), (33, 16384, 40, 1), (64, 2048, 2048, 1),
    (1024, 1024, 64, 1), (1024, 1024, 65, 2), (2000, 130, 300, 1), (130, 9000, 100, 1), (4096, 64, 1024, 1),
    (100, 4096, 1024, 1), (2048, 2048, 40, 1), (70000, 33, 128, 1), (70000, 33, 129, 1), (70000, 32, 129, 1),
    (33, 70000, 20, 1)])
@pytest.mark.parametrize("order", ["mn", "nm"])
def test_planner_choice(handle, prec, M, N, K, Z, order):
    _run(handle, prec, M, N, K, Z, order)


@pytest.mark.parametrize("prec", ["fp64", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("rows", [32, 64, 96, 128, 100])
@pytest.mark.parametrize("K", [40, 300])
def test_planned_mask(handle, prec, rows, K):
    """Rows of a skipped item stay as they were wherever some tile fits the item."""
    import torch
    td = torch.complex128 if prec == "fp64" else torch.complex64
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    A = torch.randn((64, rows, K), generator=g, dtype=td, device="cuda")
    B = torch.randn((K, 300), generator=g, dtype=td, device="cuda")
    C = torch.full((64, rows, 300), 5.0, dtype=td, device="cuda")
    mask = (torch.arange(64, device="cuda") % 3 != 0).to(torch.int32)
    handle.test_contract(prec, "zak", A, "kc", B, "zac", C, mask=mask)
    a, b = A.to(torch.complex128).cpu(), B.to(torch.complex128).cpu()
    err = (C.to(torch.complex128).cpu() - a @ b).abs() / (a.abs() @ b.abs())
    on = mask.cpu().bool()
    assert float(err[on].max()) < TOL[prec]
    if rows % 32 == 0:
        assert bool((C[~on.cuda()] == 5.0).all())
    else:
        assert float(err.max()) < TOL[prec]


@pytest.mark.parametrize("prec", ["bf16x3", "bf16x6"])
@pytest.mark.parametrize("eq", ["zak,zkc,zac", "zak,kc,zac", "ak,zkc,azc", "zqak,zqkc,zqac"])
@pytest.mark.parametrize("kept", ["some", "none"])
def test_packed_mask(handle, prec, eq, kept):
    """What the packing of a masked launch leaves out is never read: kept items
    are right, skipped ones as they were (packed operands; K leaves a remainder)."""
    import torch
    ia, ib, ic = eq.split(",")
    dim = dict(z=6, q=2, a=320, c=320, k=200)
    g = torch.Generator(device="cuda").manual_seed(len(eq))
    A, B = (torch.randn([dim[l] for l in i], generator=g, dtype=torch.complex64, device="cuda") for i in (ia, ib))
    C = torch.full([dim[l] for l in ic], 5.0, dtype=torch.complex64, device="cuda")
    on = torch.tensor([1, 0, 1, 1, 0, 0] if kept == "some" else [0] * 6).bool()
    handle.test_contract(prec, ia, A, ib, B, ic, C, mask=on.to(torch.int32).cuda(), cfg=0)
    a, b = A.to(torch.complex128).cpu(), B.to(torch.complex128).cpu()
    err = (C.to(torch.complex128).cpu() - torch.einsum(f"{ia},{ib}->{ic}", a, b)).abs()
    err = (err / torch.einsum(f"{ia},{ib}->{ic}", a.abs(), b.abs())).movedim(ic.index("z"), 0)
    got = C.cpu().movedim(ic.index("z"), 0)
    assert bool((got[~on] == 5.0).all())
    assert kept == "none" or float(err[on].max()) < TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("M,N,K,Z", [(1, 1, 1, 1), (15, 17, 3, 2), (16, 16, 16, 3), (33, 16, 17, 300), (16, 40, 65, 1),
                                     (17, 5, 129, 2), (40, 33, 257, 1), (1, 70, 2100, 1)])
@pytest.mark.parametrize("ksplit", [1, 3])
@pytest.mark.parametrize("eq", ["zmk,zkn,zmn", "zkm,znk,znm"])
def test_wave_tile(handle, prec, M, N, K, Z, ksplit, eq):
    """The 16x16 tile, whose waves share K: fewer k than waves, remainders of a
    quad and of a batch of quads, either operand contiguous along k."""
    import torch
    td = torch.complex128 if prec == "fp64" else torch.complex64
    dim = dict(z=Z, m=M, n=N, k=K)
    ia, ib, ic = eq.split(",")
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    A, B = (torch.randn([dim[l] for l in i], generator=g, dtype=td, device="cuda") for i in (ia, ib))
    C = torch.randn([dim[l] for l in ic], generator=g, dtype=td, device="cuda")
    a, b, c = (x.to(torch.complex128).cpu() for x in (A, B, C))
    handle.test_contract(prec, ia, A, ib, B, ic, C, conjB=True, accumulate=True, cfg=7, ksplit=ksplit)
    ref = c + torch.einsum(f"{ia},{ib}->{ic}", a, b.conj().resolve_conj())
    scale = c.abs() + torch.einsum(f"{ia},{ib}->{ic}", a.abs(), b.abs())
    assert float(((C.to(torch.complex128).cpu() - ref).abs() / scale).max()) < TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("ksplit", [1, 2])
def test_wave_tile_tables(handle, prec, ksplit):
    """K offsets that no stride gives, and a masked launch with items of 16 rows."""
    import torch
    td = torch.complex128 if prec == "fp64" else torch.complex64
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randn((12, 7, 16, 13), generator=g, dtype=td, device="cuda")  # z j m l
    B = torch.randn((13, 21, 7), generator=g, dtype=td, device="cuda")      # l n j
    C = torch.full((12, 16, 21), 5.0, dtype=td, device="cuda")
    mask = (torch.arange(12, device="cuda") % 3 != 1).to(torch.int32)
    handle.test_contract(prec, "zjml", A, "lnj", B, "zmn", C, cfg=7, ksplit=ksplit, mask=mask)
    a, b = A.to(torch.complex128).cpu(), B.to(torch.complex128).cpu()
    err = (C.to(torch.complex128).cpu() - torch.einsum("zjml,lnj->zmn", a, b)).abs()
    err = err / torch.einsum("zjml,lnj->zmn", a.abs(), b.abs())
    on = mask.cpu().bool()
    assert float(err[on].max()) < TOL[prec]
    assert bool((C.cpu()[~on] == 5.0).all())
