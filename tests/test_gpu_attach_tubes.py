"""Tubes are searched 16 tracks to a block, a lane per track and row: track
counts around a block and tubes from none to every row, against the oracle
cluster by cluster."""
import numpy as np
import pytest

import synth
from gpu_common import run_gpu
from test_gpu_attach import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tracks", [1, 15, 18, 20, 34, 36, 70])
@pytest.mark.parametrize("radius", [0.05, 1.5, 40.0])
def test_tubes(n_tracks, radius):
    ev = synth.make_config1(n_tracks=n_tracks)
    g, track, state = _check(ev, radius=radius)
    print(n_tracks, "tracks", g["status"]["n_tracks"], flush=True)


def test_no_tracks():
    ev = synth.make_config1(n_tracks=3)
    keep = ev.row < 8          # too few rows for a track
    import dataclasses
    n = int(keep.sum())
    ev = dataclasses.replace(ev, sector_offsets=np.array([0, n], np.int64),
                             **{f: getattr(ev, f)[keep]
                                for f in ("row", "y", "z", "charge", "label")})
    _, g = run_gpu(ev)
    assert g["status"]["n_tracks"] == 0
    _, track, state = _check(ev)
    assert (track == -1).all() and not state.any()
