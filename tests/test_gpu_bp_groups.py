"""Belief propagation where its grouped contractions change tiles or slices, one
sweep at a time against the oracle's update: bonds on both sides of the 16
columns of the narrow tile, sums of one entry (legs without a bond), sums cut
into K slices, and sums longer than one k table (1024 entries).

One sweep from the identity has one rounding chain per message, so the messages
agree to a few hundred unit roundoffs of their unit norm: 1e-13."""
import numpy as np
import pytest

from peps_inputs import brick_lattice, heavy_hex_lattice, random_peps, square_lattice
from oracle import bp as obp

pytestmark = pytest.mark.gpu

STATES = {
    "pair_D1": lambda: square_lattice(1, 2, 1),
    "chain_D16": lambda: square_lattice(1, 4, 16),
    "chain_D33": lambda: square_lattice(1, 4, 33),
    "brick_D17": lambda: brick_lattice(3, 4, 17),
    "heavyhex_D16": lambda: heavy_hex_lattice(2, 5, 16),
    "heavyhex_D24": lambda: heavy_hex_lattice(2, 5, 24),
    "square_D12": lambda: square_lattice(3, 3, 12),
}


@pytest.mark.parametrize("name", list(STATES))
@pytest.mark.parametrize("sweeps", [1, 3])
def test_bp_sweeps_match_oracle(name, sweeps):
    import paper_2507_11424_amd as tnb
    lat = STATES[name]()
    T = random_peps(lat, "haar", 0.3, 71)
    M, _, _ = obp.bp_messages(T, max_iter=sweeps, tol=0.0)
    h = tnb.Handle(0)
    try:
        got = h.bp(tnb.Peps.from_numpy(lat, T), max_sweeps=sweeps, tol=0.0, loops=False, want_messages=True)
    finally:
        h.close()
    assert got["sweeps"] == sweeps
    m = got["messages"].cpu().numpy()
    for (r, c, leg), ref in M.items():
        d = ref.shape[0]
        block = m[r * lat.cols + c, leg - 1]
        assert np.abs(block[:d, :d] - ref).max() < 1e-13, (r, c, leg)
        assert np.all(block[d:] == 0) and np.all(block[:, d:] == 0)
