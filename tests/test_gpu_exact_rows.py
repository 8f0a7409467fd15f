"""Exact boundary rows whose site matrices are tall (D^2 columns above 16, D^4
rows above 128), where the canonical form takes CholeskyQR with R = Q^H A and, for
a rank-deficient site, the Householder tree: the norm of a two-row state against
the oracle, for full-rank, graded and rank-deficient bonds."""
import pytest

from peps_inputs import random_peps, square_lattice
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [4, 5, 8])
@pytest.mark.parametrize("bond", ["full", "graded", "deficient"])
@pytest.mark.parametrize("dtype,prec,tol", [("c128", "fp64", 1e-10), ("c64", "fp32", 1e-3)])
def test_exact_rows(D, bond, dtype, prec, tol):
    import numpy as np
    import paper_2507_11424_amd as tnb
    lat = square_lattice(2, 3, D)
    T = random_peps(lat, "haar", 0.6, 100 + D)
    if bond != "full":
        w = np.logspace(0, -9, D) if bond == "graded" else np.r_[np.ones(D // 2), np.zeros(D - D // 2)]
        for row in T:
            for c in range(2):
                row[c] = row[c] * w  # the right leg is the last
    if dtype == "c64":
        T = [[t.astype(np.complex64).astype(np.complex128) for t in row] for row in T]
    ref = oracle.norm(T, 64, sweeps=2, seed=0, direction=0)
    h = tnb.Handle(0)
    try:
        got = h.boundary_contract(tnb.Peps.from_numpy(lat, T, dtype=dtype), tnb.make_opts(chi=64, prec=prec))
    finally:
        h.close()
    assert abs(got[0] - ref[0]) < tol, (got, ref)
    assert abs(got[1] - ref[1]) < tol
