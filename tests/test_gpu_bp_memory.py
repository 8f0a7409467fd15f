"""Belief propagation in little memory: where the intermediates of a stage do not fit
together it contracts them one after another, and the intermediates of the sweeps are
gone before those of the loops come.

The 4x4 lattice at D = 8 has 0.66 MiB of sites (complex128), staged and gathered by
shape; a sweep's intermediates together are eight times that, those of the loops'
four leg pairs again eight, beside the pair tensors (4.2 MiB) and, later, the loop
matrices (2.3 MiB and two products of 0.6)."""
import numpy as np
import pytest

from peps_inputs import random_peps, square_lattice

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _bp(cap, loops):
    import paper_2507_11424_amd as tnb
    lat = square_lattice(4, 4, 8)
    peps = tnb.Peps.from_numpy(lat, random_peps(lat, "haar", 0.3, 31))
    h = tnb.Handle(0)
    try:
        h.test_workspace(cap)
        r = h.bp(peps, loops=loops, want_messages=True)
        assert h.test_workspace(0) == 0  # everything given back
    finally:
        h.close()
    return r


# without loops: one after another in 4 MiB, together in 8; with loops: 12 MiB hold the
# loops' stage together once the sweeps' buffers are gone (16 with them: 17 and more)
@pytest.mark.parametrize("cap,loops", [(4, False), (8, False), (12, True), (16, True)])
def test_capped(cap, loops):
    want, got = _bp(0, loops), _bp(cap * MIB, loops)
    assert got["sweeps"] == want["sweeps"]
    assert abs(got["log_abs_Z"] - want["log_abs_Z"]) < 1e-11
    assert float((got["messages"] - want["messages"]).abs().max()) < 1e-12
    if loops:
        assert np.abs(got["eps_loops"] - want["eps_loops"]).max() < 1e-11


def test_too_little():
    """What does not fit either way is still an out-of-memory error, and the handle
    serves the next call."""
    import paper_2507_11424_amd as tnb
    lat = square_lattice(4, 4, 8)
    peps = tnb.Peps.from_numpy(lat, random_peps(lat, "haar", 0.3, 31))
    h = tnb.Handle(0)
    try:
        h.test_workspace(2 * MIB)
        with pytest.raises(tnb.TnError) as e:
            h.bp(peps, loops=False)
        assert e.value.status == 3
        h.test_workspace(0)
        assert h.bp(peps, loops=False)["sweeps"] > 1
    finally:
        h.close()
