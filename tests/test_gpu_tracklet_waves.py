"""Tracklet construction deals the starts to waves by their count: one to a
wave, a few, or 64.  Parity with the oracle (equality of bits) at counts that
put one, a few and some dozens of them in a wave (145 to 12,000 starts), and
with starts beyond the capacity cut off alike."""
import numpy as np
import pytest

import synth
from gpu_common import assert_same_tracking, run_gpu, run_oracle, same_floats

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_primary", [60, 500, 1100, 2000, 4000])
def test_parity_by_start_count(n_primary):
    ev = synth.make_config2(seed=5, n_primary=n_primary)
    _, g = run_gpu(ev)
    print("starts", g["status"]["n_starts"], flush=True)
    assert_same_tracking(g, run_oracle(ev), ev.n_clusters)


@pytest.mark.parametrize("cap", [1, 63, 65, 700])
def test_capacity_below_the_start_count(cap):
    """The tracklets below the capacity are those of the full run."""
    ev = synth.make_config2(seed=5, n_primary=500).sector(4)
    _, full = run_gpu(ev)
    _, g = run_gpu(ev, start_capacity=cap)
    n = min(cap, full["t_start"].shape[0])
    assert g["t_start"].shape[0] == n
    for k in ("t_start", "t_hits", "t_nhits", "t_rin"):
        assert np.array_equal(g[k], full[k][:n]), k
    for k in ("t_par", "t_cov", "t_chi2"):
        assert same_floats(g[k], full[k][:n]), k
