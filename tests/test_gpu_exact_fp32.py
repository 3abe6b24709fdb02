"""The short reciprocal, square root and division of the Kalman kernels equal
the correctly rounded operators bit for bit: every float of the range they
are used on (reciprocal and root), eight numerators for every denominator
(division); and the tracklets built with them equal the oracle's.  No
tolerance: equality of bits."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth
from gpu_common import run_gpu, run_oracle, same_floats, to_ids
from paper_1905_05515_amd import _lib as L

pytestmark = pytest.mark.gpu


def bits(v):
    return int(np.float32(v).view(np.uint32))


@pytest.mark.parametrize("op,lo,hi", [
    (0, bits(2.0 ** -125), bits(2.0 ** 125) + 1),       # 1 / b, positive
    (0, bits(-(2.0 ** -125)), bits(-(2.0 ** 125)) + 1),  # and negative
    (1, bits(2.0 ** -100), bits(2.0 ** 120) + 1),       # sqrt
    (2, 0, 0x7F800001),                                 # any 1 / b, infinity included
    (2, 0x80000000, 0xFF800001),
    (3, bits(2.0 ** -20), bits(2.0 ** 20) + 1),         # a / b
])
def test_equal_to_the_correctly_rounded_operator(op, lo, hi):
    bad = torch.zeros(1, dtype=torch.int64, device="cuda")
    L.check(L.lib().tpc_check_exact_fp32(op, lo, hi, C.c_void_p(bad.data_ptr()),
                                         C.c_void_p(torch.cuda.current_stream().cuda_stream)),
            "tpc_check_exact_fp32")
    assert int(bad.item()) == 0


@pytest.mark.parametrize("s_max", [0.5, 1.0, 1.05])
def test_tracklets_on_both_sides_of_the_range_rule(s_max):
    """The transport takes the short sequences up to s_max = 1 and the general
    operators beyond: tracklets equal to the oracle's bit for bit."""
    ev = synth.make_config1(seed=11, n_tracks=30)
    prm = dict(synth.default_params(), s_max=s_max)
    _, g = run_gpu(ev, prm=prm)
    o = run_oracle(ev, prm=prm)["tracklets"]
    assert np.array_equal(to_ids(g, ev.n_clusters)["hits"], o["hits"])
    assert np.array_equal(g["t_nhits"], o["nhits"])
    for k in ("par", "cov", "chi2"):
        assert same_floats(g["t_" + k], o[k]), k
