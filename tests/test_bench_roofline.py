"""Bytes per hit that the bench prices the refit kernels at: they follow the
library's rule for the states it keeps."""
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def test_line_is_the_librarys():
    import bench
    src = open(os.path.join(ROOT, "paper_1905_05515_amd", "csrc", "refit.hip")).read()
    bits = re.search(r"kSparseTracks = int64_t\(1\) << (\d+);", src).group(1)
    assert bench.REFIT_SPARSE_TRACKS == 1 << int(bits)


@pytest.mark.parametrize("kernel,tracks,per_hit", [
    ("k_refit_fwd<tpc::kPacked>", 65535, 89), ("k_refit_fwd<tpc::kPacked>", 65536, 49),
    ("k_refit_adj<1>", 65535, 97), ("k_refit_adj<2>", 65536, 57), ("k_refit_pack", 400, 18)])
def test_bytes_per_hit(kernel, tracks, per_hit):
    import bench
    r = bench.roofline(kernel, 1.0, {}, 1000, 5000, tracks)
    assert r["algorithmic_bytes_per_unit"] == per_hit
    assert r["achieved"] == pytest.approx(per_hit * 5000 / 1e-3 / 1e9)
