"""Grid buckets (a pad row's z slab) around the sizes where their sorting
changes: in one block's LDS up to 1024 clusters, in a compute unit's up to
16128, dealt in two passes beyond.  One row of the sector, or its invalid
rows, hold that many; equality with the form that runs as one launch, which
deals every bucket."""
import dataclasses

import numpy as np
import pytest

import synth
from gpu_common import run_gpu

pytestmark = pytest.mark.gpu
KEYS = ("bin_start", "idg", "yg", "zg", "starts", "t_hits", "trk_hits")


@pytest.mark.parametrize("n", [1024, 1025, 4097, 16128, 16129, 40000])
@pytest.mark.parametrize("row", [70, 255])
@pytest.mark.parametrize("large", [False, True])
def test_bucket_sizes(n, row, large):
    """large: more than 512 clusters in the other rows too."""
    ev = synth.make_config1()
    if large:
        h = synth.make_config2(seed=5, n_primary=2000).sector(4)
        k = 10
        rep = {f: np.concatenate([getattr(ev, f)] + [getattr(h, f)] * k)
               for f in ("row", "y", "z", "charge", "label")}
        ev = dataclasses.replace(ev, sector_offsets=np.array([0, len(rep["row"])], np.int64),
                                 **rep)
    g = np.random.Generator(np.random.PCG64(n))
    keep = ev.row != row
    add = dict(row=np.full(n, row), y=g.uniform(-20, 20, n), z=g.uniform(0, 250, n),
               charge=np.ones(n), label=np.full(n, -1))
    order = g.permutation(int(keep.sum()) + n)
    rep = {f: np.concatenate([getattr(ev, f)[keep], add[f].astype(getattr(ev, f).dtype)])[order]
           for f in add}
    ev = dataclasses.replace(ev, sector_offsets=np.array([0, order.size], np.int64), **rep)
    a, b = (run_gpu(ev, mode=m)[1] for m in ("staged", "persistent"))
    assert a["status"]["n_grid"] == order.size
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), k
