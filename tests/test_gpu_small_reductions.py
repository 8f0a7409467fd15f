"""Norms, normalisation and dot products at the sizes where their launches
change: two sites joined by one bond of dimension D, so that the reduced vectors
have D^2 entries (2048 and 8192: one workgroup's registers; above, parts of 16-byte words
where those tile the vector)."""
import math

import numpy as np
import pytest

from peps_inputs import square_lattice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [1, 45, 46, 90, 91, 128, 129, 600])
@pytest.mark.parametrize("dtype,prec,tol", [("c128", "fp64", 1e-11), ("c64", "fp32", 1e-4)])
def test_two_sites(D, dtype, prec, tol):
    import torch
    import paper_2507_11424_amd as tnb
    rng = np.random.default_rng(D)
    lat = square_lattice(1, 2, D)
    T = [rng.uniform(0.1, 1, (2, D)) + 1j * rng.uniform(-0.2, 0.2, (2, D)) for _ in range(2)]
    if dtype == "c64":
        T = [t.astype(np.complex64).astype(np.complex128) for t in T]
    peps = tnb.Peps.from_numpy(lat, [[T[0].reshape(2, 1, 1, 1, D), T[1].reshape(2, 1, D, 1, 1)]], dtype=dtype)
    p = np.abs(np.einsum("sb,tb->st", T[0], T[1])) ** 2
    h = tnb.Handle(0)
    try:
        o = tnb.make_opts(chi=4, prec=prec)
        got = h.boundary_contract(peps, o)
        bits, lq, lp = h.sample(peps, o, 24, seed=3)[:3]
        torch.cuda.synchronize()
    finally:
        h.close()
    assert abs(got[0] - math.log(p.sum())) < tol
    assert abs(got[1]) < tol
    b = bits.cpu().numpy()
    want = np.log(p[b[:, 0], b[:, 1]])
    assert np.abs(lq.cpu().numpy() - (want - math.log(p.sum()))).max() < tol
    assert np.abs(lp.cpu().numpy() - want).max() < tol
