"""The timing report names kernels as they are called: no namespace, whole
template arguments, no stray parenthesis."""
import re

import pytest

import synth
from gpu_common import ctx, run_gpu
from paper_1905_05515_amd import api

pytestmark = pytest.mark.gpu


def test_names_of_the_timing_report():
    ev = synth.make_config1()
    api.timing_enable(ctx(), True)
    try:
        run_gpu(ev)
        names = set(api.timing_report(ctx()))
    finally:
        api.timing_enable(ctx(), False)
    assert "k_tracklets" in names and any(n.startswith("k_scan_tiles<") for n in names)
    for n in names:
        assert re.fullmatch(r"k_\w+(<[^()<>]*>)?", n), n
