"""Big sectors (131072 clusters and more) process their starts by z slab and
row, in groups of at most 65536, and put the hit lists back in order.  One
group, several, a row too long for the 16-bit offsets (no order then), a big
sector between small ones, a start capacity that cuts a group.  The
persistent form keeps the order of the starts: equality of every output."""
import dataclasses

import numpy as np
import pytest

import synth
from gpu_common import run_gpu, same_floats

pytestmark = pytest.mark.gpu
INTS = ("starts", "t_start", "t_nhits", "t_rin", "t_hits", "trk_off", "trk_hits", "trk_tracklet")
FLOATS = ("t_par", "t_cov", "t_chi2")


def stacked(k, per=20.0):
    """One sector with k copies of a central event's, one behind the other in z."""
    ev = synth.make_config2(seed=5, n_primary=2000).sector(4)
    z0, z1 = ev.sector_range[0, 2:4]
    rep = {f: np.concatenate([getattr(ev, f)] * k) for f in ("row", "y", "charge", "label")}
    z = np.concatenate([(ev.z + np.float32(per * i)).astype(np.float32) for i in range(k)])
    rng = ev.sector_range.copy()
    rng[0, 3] = z1 + per * (k - 1)
    return dataclasses.replace(ev, z=z, sector_range=rng,
                               sector_offsets=np.array([0, z.shape[0]], np.int64), **rep)


def with_long_row(ev, n=66000, row=70):
    """n more clusters on one row, spread over the sector."""
    g = np.random.Generator(np.random.PCG64(2))
    y0, y1, z0, z1 = ev.sector_range[0]
    add = dict(row=np.full(n, row, ev.row.dtype), y=g.uniform(y0 * .5, y1 * .5, n),
               z=g.uniform(z0, z1, n), charge=np.ones(n), label=np.full(n, -1))
    rep = {f: np.concatenate([getattr(ev, f), add[f].astype(getattr(ev, f).dtype)]) for f in add}
    return dataclasses.replace(ev, sector_offsets=np.array([0, rep["row"].shape[0]], np.int64),
                               **rep)


def joined(evs):
    off = np.cumsum([0] + [e.n_clusters for e in evs]).astype(np.int64)
    rep = {f: np.concatenate([getattr(e, f) for e in evs])
           for f in ("row", "y", "z", "charge", "label", "sector_range", "sector_side")}
    return dataclasses.replace(evs[0], sector_offsets=off, **rep)


def make(kind):
    if kind == "one_group":
        return stacked(14)
    if kind == "groups":
        return stacked(240)
    if kind == "long_row":
        return with_long_row(stacked(14))
    small = synth.make_config2(seed=6, n_primary=2000)
    k = dict(mixed=[15], around_the_line=[9, 10, 11])[kind]
    return joined([small.sector(3)] + [stacked(i) for i in k] + [small.sector(5)])


@pytest.mark.parametrize("kind,cap", [("one_group", None), ("groups", None), ("long_row", None),
                                      ("mixed", None), ("one_group", 3001), ("mixed", 2500)])
def test_same_as_the_order_of_the_starts(kind, cap):
    ev = make(kind)
    kw = {} if cap is None else dict(start_capacity=cap)
    sizes = np.diff(ev.sector_offsets)
    assert sizes.max() >= 1 << 17
    res = {}
    for mode in ("staged", "persistent"):
        res[mode] = run_gpu(ev, mode=mode, **kw)[1]
        s = res[mode]["status"]
        print(kind, mode, sizes, s["n_starts"], s["n_tracks"], flush=True)
    a, b = res["staged"], res["persistent"]
    if kind == "groups":
        assert a["status"]["n_starts"] > 65536
    if cap is not None:
        assert a["status"]["n_starts"] > cap
    for k in INTS:
        assert np.array_equal(a[k], b[k]), k
    for k in FLOATS:
        assert same_floats(a[k], b[k]), k
    for k in ("n_propagations", "n_updates", "n_candidates", "n_starts", "n_tracks"):
        assert a["status"][k] == b["status"][k], k
    # the stages called one by one, too
    if cap is None:
        c = run_gpu(ev)[1]
        for k in INTS:
            assert np.array_equal(a[k], c[k]), k


def test_selection_forms_side_by_side():
    """Sectors of 86,000, 95,000 and 105,000 clusters between small ones: the
    larger two select by row, the others by chunk; their tracklets share words
    of the kept bits.  Every form gives the same tracks."""
    ev = make("around_the_line")
    print(np.diff(ev.sector_offsets), flush=True)
    a = run_gpu(ev, mode="persistent")[1]
    for mode in ("staged", "per_sector"):
        b = run_gpu(ev, mode=mode)[1]
        for k in INTS:
            assert np.array_equal(a[k], b[k]), (mode, k)
