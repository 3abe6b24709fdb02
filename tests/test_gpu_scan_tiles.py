"""Compaction of starts and tracks over tiles of 2048: one tile, its edges,
several tiles, and more than 1024 of them, where the tile sums are scanned by
a launch of their own instead of by the tiles.  The persistent form counts
sector by sector and shares none of it: equality of every output; the oracle
at the sizes it takes."""
import dataclasses

import numpy as np
import pytest

import synth
from gpu_common import assert_same_tracking, run_gpu, run_oracle

pytestmark = pytest.mark.gpu
KEYS = ("starts", "t_start", "t_nhits", "t_hits", "trk_off", "trk_hits", "trk_tracklet")
COUNTS = ("n_starts", "n_tracks", "n_track_hits", "overflow")


def copies(ev, k):
    """k copies of the event's sectors, one after the other."""
    n = ev.n_clusters
    off = np.concatenate([ev.sector_offsets[:-1] + i * n for i in range(k)] + [[k * n]])
    rep = {f: np.concatenate([getattr(ev, f)] * k)
           for f in ("row", "y", "z", "charge", "label", "sector_range", "sector_side")}
    return dataclasses.replace(ev, sector_offsets=off.astype(np.int64), **rep)


def cut(ev, n):
    """The first n clusters of a one-sector event."""
    rep = {f: getattr(ev, f)[:n] for f in ("row", "y", "z", "charge", "label")}
    return dataclasses.replace(ev, sector_offsets=np.array([0, n], np.int64), **rep)


@pytest.mark.parametrize("n", [1, 2, 2047, 2048, 2049, 4096, 4097, 6150])
def test_parity_around_tile_edges(n):
    ev = cut(synth.make_config2(seed=5, n_primary=2000).sector(4), n)
    assert ev.n_clusters == n
    _, g = run_gpu(ev)
    assert_same_tracking(g, run_oracle(ev), n)


@pytest.mark.parametrize("tiles", [900, 1025, 3100])
def test_forms_agree_on_many_tiles(tiles):
    """At least so many tiles of clusters; a third as many of start capacity."""
    ev = synth.make_config2(seed=5, n_primary=1100)
    ev = copies(ev, tiles * 2048 // ev.n_clusters + 1)
    res = {}
    for mode in ("staged", "persistent"):
        print(mode, ev.n_clusters, ev.n_sectors, flush=True)
        res[mode] = run_gpu(ev, mode=mode)[1]
    a, b = res["staged"], res["persistent"]
    for k in COUNTS:
        assert a["status"][k] == b["status"][k], k
    assert a["status"]["n_tracks"] > 0
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), k
