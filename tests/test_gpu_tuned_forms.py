"""What the tuner may put in a mode's place: in the split-BF16 modes the FP32 kernel
with four real products, never the one with three. In a saved file the last number
of a line says it: 0 the mode's own kernel, 2 four products (1: three, from older
files, still read)."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(262144, 64, 40, 1), (131072, 32, 48, 2), (65536, 16, 64, 1), (4096, 1, 100, 1), (100, 90, 40, 20),
          (64, 64, 300, 1), (1000, 48, 33, 3), (16384, 128, 64, 1)]


@pytest.mark.parametrize("prec", ["bf16x3", "bf16x6"])
def test_split_modes(prec, tmp_path):
    import torch
    import paper_2507_11424_amd as tnb
    path = tmp_path / "tuned.txt"
    h = tnb.Handle(0)
    try:
        h.set_autotune(True, str(path))
        for M, N, K, Z in SHAPES:
            g = torch.Generator(device="cuda").manual_seed(M + N + K)
            A = torch.randn((Z, M, K), generator=g, dtype=torch.complex64, device="cuda")
            B = torch.randn((Z, K, N), generator=g, dtype=torch.complex64, device="cuda")
            C = torch.empty((Z, M, N), dtype=torch.complex64, device="cuda")
            h.test_contract(prec, "zmk", A, "zkn", B, "zmn", C)
        torch.cuda.synchronize()
    finally:
        h.close()
    forms = [int(l.split()[-1]) for l in path.read_text().splitlines()]
    assert len(forms) == len(SHAPES)
    assert set(forms) <= {0, 2}, forms


@pytest.mark.parametrize("prec", ["fp64", "bf16x6"])
@pytest.mark.parametrize("form,cfg", [(1, 0), (2, 0), (2, 1), (2, 2), (2, 5), (2, 7), (2, 8), (2, 3), (2, 4), (2, 6)])
def test_saved_forms(prec, form, cfg, tmp_path):
    """Every entry that a file may hold runs; one of a tile that the four products do
    not have is not taken."""
    import torch
    import paper_2507_11424_amd as tnb
    path = tmp_path / "tuned.txt"
    td = torch.complex128 if prec == "fp64" else torch.complex64
    g = torch.Generator(device="cuda").manual_seed(cfg)
    A = torch.randn((300, 70), generator=g, dtype=td, device="cuda")
    B = torch.randn((70, 150), generator=g, dtype=td, device="cuda")
    C = torch.empty((300, 150), dtype=td, device="cuda")
    for write in (True, False):
        h = tnb.Handle(0)
        try:
            h.set_autotune(True, str(path))
            h.test_contract(prec, "mk", A, "kn", B, "mn", C)
            torch.cuda.synchronize()
        finally:
            h.close()
        if write:
            key = path.read_text().splitlines()[0].split()[0]
            path.write_text(f"{key} {cfg} 1 0 {form}\n")
    a, b = A.to(torch.complex128).cpu(), B.to(torch.complex128).cpu()
    err = ((C.to(torch.complex128).cpu() - a @ b).abs() / (a.abs() @ b.abs())).max()
    # sums of 70 terms of four products, two roundings each
    assert float(err) < 4 * 70 * 2.0 ** (-53 if prec == "fp64" else -24)
