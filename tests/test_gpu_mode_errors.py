"""Errors of the reduced modes against 64 bits: sums that bf16x6 hands to the FP32
kernel are no further off than those of its own kernel (root mean square over many
sums, five per cent for chance), and FP32 log-norms and probabilities of small exact
states agree with 64 bits to 1e-5."""
import math

import numpy as np
import pytest

from peps_inputs import random_peps, square_lattice
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 5, 8, 16, 24, 32])
@pytest.mark.parametrize("M,N", [(20000, 64), (4096, 24), (300, 200)])
@pytest.mark.parametrize("positive", [False, True])
def test_bf16x6_short_sums(M, N, K, positive):
    import torch
    import paper_2507_11424_amd as tnb
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    A = torch.randn((M, K), generator=g, dtype=torch.complex64, device="cuda")
    B = torch.randn((K, N), generator=g, dtype=torch.complex64, device="cuda")
    if positive:
        A, B = (torch.complex(x.real.abs(), x.imag.abs()) for x in (A, B))
    a, b = A.cpu().to(torch.complex128), B.cpu().to(torch.complex128)
    want, scale = a @ b, a.abs() @ b.abs()
    rms = []
    h = tnb.Handle(0)
    try:
        for cfg in (-1, 0):  # the planner's choice; the split kernel
            C = torch.empty((M, N), dtype=torch.complex64, device="cuda")
            h.test_contract("bf16x6", "mk", A, "kn", B, "mn", C, cfg=cfg)
            rms.append(float(((C.cpu().to(torch.complex128) - want).abs() / scale).square().mean().sqrt()))
    finally:
        h.close()
    assert rms[0] <= 1.05 * rms[1], rms


@pytest.mark.parametrize("D", [4, 5, 8])
@pytest.mark.parametrize("bond", ["full", "graded", "deficient"])
def test_fp32_exact_rows(D, bond):
    import paper_2507_11424_amd as tnb
    lat = square_lattice(2, 3, D)
    T = random_peps(lat, "haar", 0.6, 200 + D)
    if bond != "full":
        w = np.logspace(0, -9, D) if bond == "graded" else np.r_[np.ones(D // 2), np.zeros(D - D // 2)]
        for row in T:
            for c in range(2):
                row[c] = row[c] * w
    T = [[t.astype(np.complex64).astype(np.complex128) for t in row] for row in T]
    ref = oracle.norm(T, 64, sweeps=2, seed=0, direction=0)
    h = tnb.Handle(0)
    try:
        got = h.boundary_contract(tnb.Peps.from_numpy(lat, T, dtype="c64"), tnb.make_opts(chi=64, prec="fp32"))
    finally:
        h.close()
    assert abs(got[0] - ref[0]) < 1e-5 and abs(got[1] - ref[1]) < 1e-5, (got, ref)


@pytest.mark.parametrize("D", [1, 45, 46, 90, 91, 128, 129, 600])
def test_fp32_two_sites(D):
    import torch
    import paper_2507_11424_amd as tnb
    rng = np.random.default_rng(1000 + D)
    lat = square_lattice(1, 2, D)
    T = [(rng.uniform(0.1, 1, (2, D)) + 1j * rng.uniform(-0.2, 0.2, (2, D))).astype(np.complex64) for _ in range(2)]
    peps = tnb.Peps.from_numpy(lat, [[T[0].reshape(2, 1, 1, 1, D), T[1].reshape(2, 1, D, 1, 1)]], dtype="c64")
    p = np.abs(T[0].astype(np.complex128) @ T[1].astype(np.complex128).T) ** 2
    h = tnb.Handle(0)
    try:
        o = tnb.make_opts(chi=4, prec="fp32")
        got = h.boundary_contract(peps, o)
        bits, lq, lp = h.sample(peps, o, 24, seed=3)[:3]
        torch.cuda.synchronize()
    finally:
        h.close()
    assert abs(got[0] - math.log(p.sum())) < 1e-5 and abs(got[1]) < 1e-5
    b = bits.cpu().numpy()
    want = np.log(p[b[:, 0], b[:, 1]])
    assert np.abs(lq.cpu().numpy() - (want - math.log(p.sum()))).max() < 1e-5
    assert np.abs(lp.cpu().numpy() - want).max() < 1e-5
