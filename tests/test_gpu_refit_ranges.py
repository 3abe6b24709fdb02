"""The refit's short division, y over a row's plane times tan_half, where it
may be taken and where not: every denominator of its range of either sign with
numerators over all of theirs and the special values (equality of bits with the
operator); geometries outside the range, which take the operator.  Scaling
tan_half by a power of two and the terms in v inversely changes no rounding:
the same bits in and out of the range."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth
from gpu_common import ctx
from paper_1905_05515_amd import _lib as L
from paper_1905_05515_amd import api

pytestmark = pytest.mark.gpu
PRM = synth.default_params()
V1, V2 = (4, 6, 11, 13), (7, 14)          # theta of the terms in v and u v, in v^2


def pattern(v):
    return int(np.float32(v).view(np.uint32))


@pytest.mark.parametrize("op", [3, 4])
@pytest.mark.parametrize("sign", [1, -1])
def test_quotients_of_the_range(op, sign):
    bad = torch.zeros(1, dtype=torch.int64, device="cuda")
    lo, hi = pattern(sign * 2.0 ** -20), pattern(sign * 2.0 ** 20) + 1
    L.check(L.lib().tpc_check_exact_fp32(op, lo, hi, C.c_void_p(bad.data_ptr()),
                                         C.c_void_p(torch.cuda.current_stream().cuda_stream)),
            "tpc_check_exact_fp32")
    assert int(bad.item()) == 0


def hits(rs):
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    return api.TrackHits(off=t(rs.trk_off), row=t(rs.row), y=t(rs.y), z=t(rs.z))


@pytest.mark.parametrize("scale", [-1.0, 2.0 ** 10, 2.0 ** -26, -2.0 ** -26, 2.0 ** 22])
def test_scaled_geometries(scale):
    rs = synth.make_config5(n_tracks=300)
    h, rx = hits(rs), torch.as_tensor(rs.row_x).cuda()
    cm = api.CALIB_MODEL
    g = torch.linspace(0.5, 1.5, rs.n_tracks, device="cuda")
    res = []
    for s in (1.0, scale):
        th = rs.theta_eval.astype(np.float32).copy()
        th[list(V1)] *= np.float32(s)
        th[list(V2)] *= np.float32(s * s)
        th = torch.as_tensor(th).cuda()
        m = dict(cm, tan_half=float(np.float32(cm["tan_half"]) * np.float32(s)))
        r = []
        for ck in (True, False):
            out = api.refit(ctx(), h, rx, PRM, th, checkpoints=ck, cm=m)
            r += [out[k].contiguous().view(torch.int32) for k in ("par", "cov", "chi2", "status")]
            if ck:
                assert int((out["status"] == 0).sum()) > rs.n_tracks // 2
                gy, gz, gt = api.refit_adjoint(ctx(), h, rx, PRM, th, out, g, cm=m)
                gt = gt.clone()
                gt[list(V1)] *= s
                gt[list(V2)] *= s * s
                r += [v.view(torch.int32) for v in (gy, gz, gt)]
        res.append(r)
    for a, b in zip(*res):
        assert torch.equal(a, b)


def test_a_plane_at_zero():
    """y over zero is infinite: a start there stops with the state the
    operator gives, not with NaN."""
    rs = synth.make_config5(n_tracks=300)
    n = 20
    row = np.tile(np.arange(n, dtype=np.uint8), 3)
    y = np.tile(np.linspace(1.0, 3.0, n, dtype=np.float32), 3)
    z = np.tile(np.linspace(10.0, 30.0, n, dtype=np.float32), 3)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    h = api.TrackHits(off=t(np.arange(0, 3 * n + 1, n, dtype=np.int32)), row=t(row), y=t(y), z=t(z))
    rx = rs.row_x.copy()
    rx[0] = 0.0
    th = np.zeros(16, np.float32)
    for base in (2, 9):                    # u is negative at the plane 0
        th[base + 2], th[base + 4], th[base + 5] = 0.1, -0.1, 0.1
    for ck in (True, False):
        out = api.refit(ctx(), h, t(rx), PRM, t(th), checkpoints=ck)
        assert (out["status"] == 2).all()
        assert (out["par"][:, 0] == float("inf")).all(), out["par"]
