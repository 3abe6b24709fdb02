"""How the refit reads its hits: packed by slot with checkpoints, straight
from the track list (with and without an index) without.  Tracks of every
length class of those readers (3 hits to all rows, around the chunk of 4 and
the packed parts of 64 slots), runs at every alignment, both z sides, and
tracks that are refused (short, long, a row outside the table anywhere).
The readers agree bit for bit, states and gradients; what they compute is
compared with the float64 oracle in test_gpu_refit.py."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth
from gpu_common import ctx
from paper_1905_05515_amd import api

pytestmark = pytest.mark.gpu
PRM = synth.default_params()
LENGTHS = (3, 4, 5, 6, 7, 8, 9, 15, 16, 17, 31, 33, 40, 63, 64, 65, 66, 67, 100, 127, 128, 129,
           130, 151, 152)


def cut(rs, lengths):
    """The first tracks of the set with at least the wanted length, cut to it."""
    off, rows, ys, zs, at = [0], [], [], [], 0
    n_of = np.diff(rs.trk_off)
    for n in lengths:
        while n_of[at] < n:
            at += 1
        a = rs.trk_off[at]
        rows.append(rs.row[a:a + n])
        ys.append(rs.y[a:a + n])
        zs.append(rs.z[a:a + n])
        off.append(off[-1] + n)
        at += 1
    return (np.array(off, np.int32), np.concatenate(rows), np.concatenate(ys),
            np.concatenate(zs))


def hits(off, row, y, z, side, gather):
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    idx = None
    if gather:
        p = np.random.Generator(np.random.PCG64(3)).permutation(row.shape[0])
        idx = np.empty(p.shape[0], np.int32)
        idx[p] = np.arange(p.shape[0], dtype=np.int32)
        row, y, z, idx = row[p], y[p], z[p], t(idx)
    return api.TrackHits(off=t(off), row=t(row), y=t(y), z=t(z), side=t(side), idx=idx)


def bits(v):
    return v.contiguous().view(torch.int32)


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("repeat", [1, 4])
def test_readers_agree(sign, repeat):
    rs = synth.make_config5(n_tracks=2000)
    off, row, y, z = cut(rs, LENGTHS * repeat)
    n = off.shape[0] - 1
    z = (sign * z).astype(np.float32)
    side = np.full(n, sign, np.int8)
    rx, th = torch.as_tensor(rs.row_x).cuda(), torch.as_tensor(rs.theta_eval).cuda()
    g = torch.linspace(0.5, 1.5, n, device="cuda")
    res = []
    for gather in (False, True):
        h = hits(off, row, y, z, side, gather)
        for ck in (True, False):
            out = api.refit(ctx(), h, rx, PRM, th, checkpoints=ck)
            res.append([bits(out[k]) for k in ("par", "cov", "chi2", "status")])
            if ck:
                grads = api.refit_adjoint(ctx(), h, rx, PRM, th, out, g)
                res[-1] += [bits(v) for v in grads]
    for r in res[1:]:
        for a, b in zip(res[0], r):
            assert torch.equal(a, b)


@pytest.mark.parametrize("n_rows", [100, 152])
@pytest.mark.parametrize("gather", [False, True])
def test_refused_tracks(n_rows, gather):
    """Status 1 (short), 3 (a row outside the table, first hit to last) and 4
    (more hits than rows, here up to 200) beside good tracks: the same from
    every reader, refused tracks zero with zero gradients."""
    rs = synth.make_config5(n_tracks=2000)
    off, row, y, z = cut(rs, (40,) * 12)
    row = (np.arange(row.shape[0]) % 40).astype(np.uint8)
    runs = [(a, a + 40) for a in off[:-1]]
    new_off, rows, ys, zs, want = [0], [], [], [], []
    for k, (a, b) in enumerate(runs):
        r, yy, zz = row[a:b].copy(), y[a:b], z[a:b]
        s = 0
        if k in (1, 2):
            r, yy, zz, s = r[:k], yy[:k], zz[:k], 1
        elif k in (3, 4, 5):
            r[(0, 20, 39)[k - 3]] = n_rows
            s = 3
        elif k in (6, 7):
            m = (n_rows + 1, 200)[k - 6]
            r, yy, zz, s = np.resize(r, m), np.resize(yy, m), np.resize(zz, m), 4
        elif k == 8:
            r, yy, zz, s = np.resize(r, 200), np.resize(yy, 200), np.resize(zz, 200), 3
            r[199] = 255
        elif k == 9:
            r, yy, zz, s = r[:0], yy[:0], zz[:0], 1
        rows.append(r), ys.append(yy), zs.append(zz), want.append(s)
        new_off.append(new_off[-1] + len(r))
    off = np.array(new_off, np.int32)
    h = hits(off, np.concatenate(rows), np.concatenate(ys), np.concatenate(zs),
             np.ones(len(want), np.int8), gather)
    rx, th = torch.as_tensor(rs.row_x[:n_rows]).cuda(), torch.as_tensor(rs.theta_eval).cuda()
    a = api.refit(ctx(), h, rx, PRM, th)
    b = api.refit(ctx(), h, rx, PRM, th, checkpoints=False)
    st = a["status"].cpu().numpy()
    for k, w in enumerate(want):
        assert st[k] == w or (w == 0 and st[k] == 2), (k, st[k], w)
    for k in ("par", "cov", "chi2", "status"):
        assert torch.equal(bits(a[k]), bits(b[k])), k
    gy, gz, gt = api.refit_adjoint(ctx(), h, rx, PRM, th, a, torch.ones(len(want), device="cuda"))
    for k, w in enumerate(want):
        sl = slice(int(off[k]), int(off[k + 1]))
        if st[k] in (1, 3, 4):
            assert not bool(a["par"][k].any()) and not bool(a["cov"][k].any())
        if st[k]:
            assert not bool(gy[sl].any()) and not bool(gz[sl].any())
    assert bool(torch.isfinite(gt).all())


@pytest.mark.parametrize("n_tracks", [(1 << 16) - 1, 1 << 16, (1 << 16) + 37])
def test_gradients_on_both_sides_of_the_checkpoint_rule(n_tracks):
    """From 65536 tracks on every second state is a checkpoint: the same bits
    for every track as in a small set, at every length class."""
    rs = synth.make_config5(n_tracks=2000)
    off, row, y, z = cut(rs, LENGTHS)
    rx, th = torch.as_tensor(rs.row_x).cuda(), torch.as_tensor(rs.theta_eval).cuda()
    n = len(LENGTHS)
    small = hits(off, row, y, z, np.ones(n, np.int8), False)
    # the same tracks over and over
    reps = -(-n_tracks // n)
    lens = np.tile(np.diff(off), reps)[:n_tracks]
    big_off = np.zeros(n_tracks + 1, np.int32)
    big_off[1:] = np.cumsum(lens)
    m = int(big_off[-1])
    big = hits(big_off, np.tile(row, reps)[:m], np.tile(y, reps)[:m], np.tile(z, reps)[:m],
               np.ones(n_tracks, np.int8), False)
    res = []
    for h in (small, big):
        out = api.refit(ctx(), h, rx, PRM, th)
        gy, gz, _ = api.refit_adjoint(ctx(), h, rx, PRM, th, out,
                                      torch.ones(h.n_tracks, device="cuda"))
        res.append((out["par"], out["chi2"], gy, gz))
    k = off[-1]
    for a, b, w in zip(res[0], res[1], (n, n, k, k)):
        tail = b.shape[0] % w
        full = b[:b.shape[0] - tail].reshape(-1, w, *b.shape[1:])
        assert torch.equal(bits(full), bits(a).expand(full.shape))
        assert torch.equal(bits(b[b.shape[0] - tail:]), bits(a)[:tail])


@pytest.mark.parametrize("n_tracks, count", [(131072, None), (131073, None), (300000, 262145),
                                             (300000, 257), (300000, 0)])
def test_order_of_many_runs(n_tracks, count):
    """The ordering cuts the tracks into at most 512 runs of whole blocks: one
    and two blocks a run, a device count far below the capacity; lengths drawn
    at random, every track as in the reader without an order."""
    rs = synth.make_config5(n_tracks=2000)
    off, row, y, z = cut(rs, (40,))
    rng = np.random.Generator(np.random.PCG64(11))
    lens = rng.integers(1, 12, n_tracks)
    big_off = np.zeros(n_tracks + 1, np.int32)
    big_off[1:] = np.cumsum(lens)
    pos = np.arange(int(big_off[-1])) - np.repeat(big_off[:-1], lens)
    h = hits(big_off, row[pos], y[pos], z[pos], np.ones(n_tracks, np.int8), False)
    if count is not None:
        d_count = torch.tensor([count], dtype=torch.int64, device="cuda")
        h.d_count = C.c_void_p(d_count.data_ptr())
    n = n_tracks if count is None else count
    rx, th = torch.as_tensor(rs.row_x).cuda(), torch.as_tensor(rs.theta_eval).cuda()
    a = api.refit(ctx(), h, rx, PRM, th)
    b = api.refit(ctx(), h, rx, PRM, th, checkpoints=False)
    for k in ("par", "cov", "chi2", "status"):
        assert torch.equal(bits(a[k][:n]), bits(b[k][:n])), k
    gy, gz, gt = api.refit_adjoint(ctx(), h, rx, PRM, th, a,
                                   torch.ones(n_tracks, device="cuda"))
    m = int(big_off[n])
    # every track of one length has the same hits: the same gradients
    for g in (gy, gz):
        g = g[:m].cpu().numpy()
        for c in range(3, 12):
            t = np.flatnonzero(lens[:n] == c)
            at = big_off[t][:, None] + np.arange(c)[None, :]
            v = g[at].view(np.int32)
            assert (v == v[:1]).all()
            if t.size:
                assert g[at[0]].any()
    assert bool(torch.isfinite(gt).all())
    assert bool(gt.any()) == (n > 0)
