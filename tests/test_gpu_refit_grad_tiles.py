"""The adjoint's hit gradients leave a tile of 64 tracks through LDS, 16 slots
at a time, written by the lanes of other tracks: tracks of every length around
those blocks of slots side by side in one tile, and in a second, partial one,
give the bits that each track gives alone."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import ctx
from paper_1905_05515_amd import api

pytestmark = pytest.mark.gpu
LENGTHS = (3, 4, 15, 16, 17, 18, 31, 32, 33, 34, 47, 48, 49, 63, 64, 65, 79, 80, 81, 95, 96, 97,
           111, 112, 113, 127, 128, 129, 143, 144, 145, 150, 151, 152)


@pytest.mark.parametrize("n_tracks", [64, 101])
def test_mixed_lengths_in_a_tile(n_tracks):
    rs = synth.make_config5(n_tracks=3000)
    n_of = np.diff(rs.trk_off)
    rng = np.random.Generator(np.random.PCG64(5))
    lens = rng.permutation(np.resize(LENGTHS, n_tracks))
    off, pick, at = [0], [], 0
    for n in lens:
        while n_of[at] < n:
            at += 1
        pick.append(np.arange(rs.trk_off[at], rs.trk_off[at] + n))
        off.append(off[-1] + n)
        at += 1
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    prm = synth.default_params()
    rx, th = t(rs.row_x), t(rs.theta_eval)
    weight = np.linspace(0.5, 1.5, n_tracks).astype(np.float32)

    def grads(tracks):
        p = np.concatenate([pick[k] for k in tracks])
        o = np.concatenate([[0], np.cumsum(lens[tracks])]).astype(np.int32)
        h = api.TrackHits(off=t(o), row=t(rs.row[p]), y=t(rs.y[p]), z=t(rs.z[p]))
        out = api.refit(ctx(), h, rx, prm, th)
        gy, gz, _ = api.refit_adjoint(ctx(), h, rx, prm, th, out, t(weight[tracks]))
        return out["status"], gy.view(torch.int32), gz.view(torch.int32)

    status, gy, gz = grads(np.arange(n_tracks))
    assert int((status == 0).sum()) >= n_tracks // 2
    for k in range(n_tracks):
        s1, y1, z1 = grads(np.array([k]))
        assert torch.equal(s1, status[k:k + 1])
        assert torch.equal(y1, gy[off[k]:off[k + 1]]), (k, lens[k])
        assert torch.equal(z1, gz[off[k]:off[k + 1]]), (k, lens[k])


@pytest.mark.parametrize("gather", [False, True])
def test_hits_are_those_of_the_forward_pass(gather):
    """The adjoint takes rows and coordinates from the checkpoints: the same
    gradients when the caller's arrays hold something else by then."""
    rs = synth.make_config5(n_tracks=200)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    prm = synth.default_params()
    rx, th = t(rs.row_x), t(rs.theta_eval)
    idx = torch.arange(rs.n_hits, dtype=torch.int32, device="cuda") if gather else None
    h = api.TrackHits(off=t(rs.trk_off), row=t(rs.row), y=t(rs.y), z=t(rs.z), idx=idx)
    out = api.refit(ctx(), h, rx, prm, th)
    g = torch.ones(rs.n_tracks, device="cuda")
    want = [v.clone() for v in api.refit_adjoint(ctx(), h, rx, prm, th, out, g)]
    other = torch.zeros_like(h.y)
    got = api.refit_adjoint(ctx(), h, rx, prm, th, out, g, y=other, z=other)
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    for v in (h.row, h.y, h.z):
        v.zero_()
    got = api.refit_adjoint(ctx(), h, rx, prm, th, out, g)
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
