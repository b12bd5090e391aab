"""The recounted roofline fraction: a particle that the seeding estimate removes
counts the instructions of the estimate as it is compiled, where `frac` keeps the
count of an earlier one.  No GPU."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench as B  # noqa: E402


def test_recounted_fraction():
    res = [{"rays": 1000, "segments": 1500, "hits": 600, "preculled": 300}]
    rec = B.launch_record("batch_kernel<16, 1> (test)", 2.0, res, 9.5, 3.25)
    ops = 700 * 950.0 + 300 * 335.0 + 1500 * (9.5 * 40.0 + 3.25 * 45.0) - 300 * 40.0 + 600 * 225.0
    assert rec["frac_recounted"] == pytest.approx(ops / 2e-3 / (256 * 64 * 2.4e9))
    assert rec["frac_recounted"] < rec["frac"]
    plain = B.launch_record("trace", 1.0, [{"rays": 10, "segments": 12, "hits": 5}], 2.0, 1.0)
    assert plain["frac_recounted"] == pytest.approx(plain["frac"])
