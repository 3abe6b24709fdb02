"""A checkpoint buffer made for the largest set serves every smaller one: its
size never falls with the tracks or the rows, on both sides of the number of
tracks from which every second state is kept."""
import numpy as np
import pytest
import torch

import synth
from paper_1905_05515_amd import api


@pytest.mark.parametrize("n_rows", [3, 4, 63, 64, 65, 151, 152, 255])
def test_size_never_falls_with_the_tracks(n_rows):
    n = np.unique(np.concatenate([
        np.arange(0, 300), np.geomspace(300, 3e6, 400).astype(np.int64),
        np.arange(65536 - 200, 65536 + 200), np.arange(131072 - 200, 131072 + 200)]))
    size = np.array([api.checkpoint_bytes(int(k), n_rows) for k in n])
    assert (np.diff(size) >= 0).all(), n[1:][np.diff(size) < 0]


@pytest.mark.parametrize("n_tracks", [1, 64, 65535, 65536, 100000, 1000000])
def test_size_never_falls_with_the_rows(n_tracks):
    size = np.array([api.checkpoint_bytes(n_tracks, r) for r in range(3, 256)])
    assert (np.diff(size) >= 0).all()


@pytest.mark.gpu
@pytest.mark.parametrize("n_large", [65536, 100000])
def test_smaller_sets_in_the_buffer_of_a_larger_one(n_large):
    from gpu_common import ctx
    rs = synth.make_config5(n_tracks=3000)
    prm = synth.default_params()
    rx, th = torch.as_tensor(rs.row_x).cuda(), torch.as_tensor(rs.theta_eval).cuda()
    shared = torch.empty(-(-api.checkpoint_bytes(n_large, rs.row_x.shape[0]) // 4),
                         dtype=torch.float32, device="cuda")
    for n in (60000, 300, 65535):
        lens = np.resize(np.diff(rs.trk_off), n)
        off = np.zeros(n + 1, np.int32)
        off[1:] = np.cumsum(lens)
        rep = lambda a: torch.as_tensor(np.resize(a, int(off[-1]))).cuda()
        h = api.TrackHits(off=torch.as_tensor(off).cuda(), row=rep(rs.row), y=rep(rs.y),
                          z=rep(rs.z))
        g = torch.ones(n, device="cuda")
        own = api.refit(ctx(), h, rx, prm, th)
        want = api.refit_adjoint(ctx(), h, rx, prm, th, own, g)
        other = {k: torch.zeros_like(v) for k, v in own.items()}
        other["checkpoints"] = shared
        got_f = api.refit(ctx(), h, rx, prm, th, out=other)
        got = api.refit_adjoint(ctx(), h, rx, prm, th, got_f, g)
        for k in ("par", "cov", "chi2", "status"):
            assert torch.equal(got_f[k].view(torch.int32), own[k].view(torch.int32)), k
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))
