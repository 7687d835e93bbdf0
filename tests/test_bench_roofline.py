"""The bench's roofline charges a launch with the bytes it must move: a part that
takes two steps reads and writes its cells once."""
import os
import sys
import types

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_two_step_parts_are_charged_one_sweep():
    # yo_time_kernel counts what the launch's steps would move one at a time
    swept = 24e9
    steps = {p: 2 if "two_step" in name or "whole_pair" in name else 1 for p, name in enumerate(bench.PART_NAMES)}
    plan = types.SimpleNamespace(time_kernel=lambda part, n: (0.0, swept * steps[part], 1e9))
    timed = [(5.0, 3)] * len(bench.PART_NAMES)         # 24 GB in 5 ms: 0.6 of 8 TB/s
    parts = bench.part_rooflines(plan, timed, (4, 16, 512), "multiport", "none")
    assert [q["part"] for q in parts] == list(bench.PART_NAMES)
    for part, q in enumerate(parts):
        assert q["frac"] == pytest.approx(0.6) and q["bytes_per_launch"] == swept, q["part"]
        assert q["one_step_bytes_per_launch"] == swept * steps[part]
    assert bench.roofline_of(parts)["frac"] == pytest.approx(0.6)
