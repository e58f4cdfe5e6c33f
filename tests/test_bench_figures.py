"""The benchmark's traffic figure comes from a counter summary only if that summary is of the launch being timed."""
import os
import re

import pytest

import bench


def summary(cfg):
    text = open(os.path.join(bench.ROOT, "profiles", f"cfg{cfg}_hbm_traffic_counters.txt")).read()
    m = re.search(r"([0-9.]+) MB of HBM traffic per launch,\s*against ([0-9.]+) MB algorithmic", text)
    return float(m.group(1)) * 1e6, float(m.group(2)) * 1e6


@pytest.mark.parametrize("cfg", [2, 3, 4, 5])
def test_traffic_is_of_a_launch_with_the_same_bytes(cfg):
    traffic, algorithmic = summary(cfg)
    assert bench.scan_traffic_from_profile(cfg, algorithmic) == (traffic, f"profiles/cfg{cfg}_hbm_traffic_counters.txt")
    assert traffic >= algorithmic
    # a launch that reads the weight too, or no longer
    for other in (1.05, 0.95):
        assert bench.scan_traffic_from_profile(cfg, algorithmic * other) == (None, None)


def test_no_summary_no_traffic():
    assert bench.scan_traffic_from_profile(99, 1e6) == (None, None)
