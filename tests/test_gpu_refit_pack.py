"""The packing of a tile's hits by one block per 64 slots, and by one block
from 1024 tiles on: around that line, tracks that are refused for a row
outside the table in each of the parts, for more hits than rows, or for both,
between good ones; states equal to the reader that packs nothing, refused
tracks zero."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import ctx
from paper_1905_05515_amd import api

pytestmark = pytest.mark.gpu
PRM = synth.default_params()


@pytest.mark.parametrize("n_tracks", [64 * 1023, 64 * 1023 + 1, 64 * 1024 + 5])
@pytest.mark.parametrize("n_rows", [64, 100, 152])
def test_both_splits(n_tracks, n_rows):
    rs = synth.make_config5(n_tracks=400)
    n_of = np.minimum(np.diff(rs.trk_off), n_rows)
    rows, ys, zs, off, want = [], [], [], [0], []
    for k in range(200):
        a, n = rs.trk_off[k], int(n_of[k])
        r, y, z = (v[a:a + n].copy() for v in (rs.row, rs.y, rs.z))
        r -= r[0]
        s = 0
        if k % 20 == 3:                                    # a row outside, in some part
            r[min(n - 1, (0, 63, 64, 128)[k // 20 % 4])] = n_rows
            s = 3
        elif k % 20 == 7:                                  # too many hits
            m = (n_rows + 1, 200)[k // 20 % 2]
            r, y, z, s = np.resize(r, m), np.resize(y, m), np.resize(z, m), 4
        elif k % 20 == 11:                                 # both, past the rows
            r, y, z, s = np.resize(r, 200), np.resize(y, 200), np.resize(z, 200), 3
            r[199] = 255
        rows.append(r), ys.append(y), zs.append(z), want.append(s)
        off.append(off[-1] + len(r))
    lens = np.resize(np.diff(off), n_tracks)
    big = np.zeros(n_tracks + 1, np.int32)
    big[1:] = np.cumsum(lens)
    t = lambda a: torch.as_tensor(np.resize(np.concatenate(a), int(big[-1]))).cuda()
    h = api.TrackHits(off=torch.as_tensor(big).cuda(), row=t(rows), y=t(ys), z=t(zs))
    rx, th = torch.as_tensor(rs.row_x[:n_rows]).cuda(), torch.as_tensor(rs.theta_eval).cuda()
    a = api.refit(ctx(), h, rx, PRM, th)
    b = api.refit(ctx(), h, rx, PRM, th, checkpoints=False)
    for k in ("par", "cov", "chi2", "status"):
        assert torch.equal(a[k].view(torch.int32), b[k].view(torch.int32)), k
    st = a["status"].cpu().numpy()
    want = np.resize(np.array(want), n_tracks)
    assert (st[want > 0] == want[want > 0]).all()
    assert (np.isin(st[want == 0], (0, 2))).all() and (st == 0).any()
    refused = torch.as_tensor(want > 0).cuda()
    assert not bool(a["par"][refused].any()) and not bool(a["cov"][refused].any())
