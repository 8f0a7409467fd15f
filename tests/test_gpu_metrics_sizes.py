"""The sample metrics at the edges of their blocks: one sample short of and past
a block of 1024 samples, a second block, the largest block count, and qubit
counts around the 16 a workgroup takes, against a direct float64 evaluation."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 1023, 1025, 65537])
@pytest.mark.parametrize("nq", [1, 15, 17])
def test_sample_stats_block_edges(n, nq):
    import torch
    import paper_2507_11424_amd as tnb
    rng = np.random.default_rng(n + nq)
    lq = rng.normal(size=n) * 3.0 - 20.0
    lp = lq + rng.normal(size=n) * 0.5 - 4.0
    bits = rng.integers(0, 2, (n, nq)).astype(np.uint8)
    w = np.exp((lp - lq - (lp - lq).max()).astype(np.longdouble))
    h = tnb.Handle(0)
    try:
        got = h.sample_stats(torch.from_numpy(lq).cuda(), torch.from_numpy(lp).cuda(), -3.0,
                             bits=torch.from_numpy(bits).cuda())
    finally:
        h.close()
    assert abs(got["log_norm_est"] - float((lp - lq).max() + np.log(w.mean()))) < 1e-12 * 10
    assert abs(got["kld"] - float((lq - lp).astype(np.longdouble).mean() - 3.0)) < 1e-12
    ess = float(w.sum() ** 2 / (w * w).sum())
    assert abs(got["ess"] - ess) < 1e-12 * ess
    z = (w[:, None] * (1 - 2 * bits.astype(np.longdouble))).sum(0) / w.sum()
    assert np.abs(got["z_is"].cpu().numpy() - z.astype(np.float64)).max() < 1e-12
