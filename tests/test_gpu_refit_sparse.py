"""The adjoint where every second state is a checkpoint (buffers for 65536
tracks and more, whatever their count) against float64: hit and theta
gradients, and those of the objective with the beam-axis term (seeds in the
last hit's state and plane), both z sides, hits in track order and gathered,
refused tracks between; tolerances of the dense form's tests: 1e-3 of a
block's norm and of its largest entry.  Dense and sparse give the same hit
gradients bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_common import ctx
from paper_1905_05515_amd import api

pytestmark = pytest.mark.gpu
PRM = synth.default_params()
N = 3000


def data(sign):
    """The set's tracks on one z side, every 50th cut to two hits (refused)."""
    rs = synth.make_config5(n_tracks=N)
    keep = np.ones(rs.n_hits, bool)
    for k in range(0, N, 50):
        keep[rs.trk_off[k] + 2:rs.trk_off[k + 1]] = False
    off = np.concatenate([[0], np.cumsum(keep)])[rs.trk_off].astype(np.int32)
    z = (sign * rs.z[keep]).astype(np.float32)
    return rs, off, rs.row[keep], rs.y[keep], z, np.full(N, sign, np.int8)


def hits(off, row, y, z, side, gather, capacity):
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    idx = None
    if gather:
        p = np.random.Generator(np.random.PCG64(9)).permutation(row.shape[0])
        idx = np.empty(p.shape[0], np.int32)
        idx[p] = np.arange(p.shape[0], dtype=np.int32)
        row, y, z, idx = row[p], y[p], z[p], t(idx)
    off = np.concatenate([off, np.full(capacity - N, off[-1], np.int32)])
    side = np.resize(side, capacity)
    count = torch.tensor([N], dtype=torch.int64, device="cuda")
    h = api.TrackHits(off=t(off), row=t(row), y=t(y), z=t(z), side=t(side), idx=idx,
                      d_count=C.c_void_p(count.data_ptr()))
    return h, count


def close(a, b):
    a = a.double().cpu().numpy()
    return (np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b) and
            np.abs(a - b).max() <= 1e-3 * np.abs(b).max())


@pytest.mark.timeout(300)
@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("gather", [False, True])
def test_gradients_against_float64(sign, gather):
    rs, off, row, y, z, side = data(sign)
    rx, th = torch.as_tensor(rs.row_x).cuda(), torch.as_tensor(rs.theta_eval).cuda()
    th64 = rs.theta_eval.astype(np.float64)
    hit_grads = []
    for capacity in (N, 70000):
        h, count = hits(off, row, y, z, side, gather, capacity)
        out = api.refit(ctx(), h, rx, PRM, th)
        st = out["status"][:N].cpu().numpy()
        assert (st[::50] == 1).all() and (st == 0).mean() > 0.95
        ok = st == 0
        g = torch.ones(capacity, device="cuda")       # the same weights at both capacities
        g[:N] = torch.linspace(0.5, 1.5, N, device="cuda")
        gy, gz, gt = (v.clone() for v in api.refit_adjoint(ctx(), h, rx, PRM, th, out, g))
        ref = oracle.refit_adjoint64(off, row, y, z, rs.row_x, PRM, th64,
                                     g[:N].cpu().numpy().astype(np.float64) * ok, side=side)
        for name, a, b in zip("yzt", (gy, gz, gt), ref):
            assert close(a, b), (capacity, name)
        loss, gp, gx, vok, w = api.vertex_residual(ctx(), h, rx, PRM, th, out)
        one = torch.ones(capacity, device="cuda")
        sy, sz, s_t = api.refit_adjoint(ctx(), h, rx, PRM, th, out, one, grad_par=gp, grad_x=gx)
        w64 = w[:N].double().cpu().numpy()
        _, og, _, _ = oracle.calib_objective(off, row, y, z, rs.row_x, PRM, th64, w64,
                                             g=ok.astype(np.float64), side=side)
        assert close(s_t, og), (capacity, "objective")
        hit_grads.append([v.clone().view(torch.int32) for v in (gy, gz, sy, sz)])
    for a, b in zip(*hit_grads):
        assert torch.equal(a, b)
