"""The benchmark credits a kernel with the work that it does: rounds visited by the timeline kernel, none by the event kernel."""
import json
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def test_event_kernel_has_no_credit_for_rounds():
    name = bench.timeline_kernel_name(1025, 100000, 4096, False, 2)
    assert name == "event_rows_kernel"
    obj = bench.roofline_object(name, 1 << 40, 1 << 39, 20.0, 20, "config5", 1 << 33, {"credit_is_bound": False})
    for key in ("achieved", "frac", "visits", "inspected", "updated", "ops_per_visit", "frac_at_two_ops_per_visit", "issue_measured"):
        assert obj[key] is None
    assert obj["hbm"]["achieved_GBps"] > 0 and json.dumps(obj)


def test_timeline_kernel_is_credited_with_its_rounds():
    name = bench.timeline_kernel_name(16384, 2000, 2048, True, 900)
    obj = bench.roofline_object(name, 1 << 40, 1 << 39, 20.0, 20, "config3", 1 << 33)
    assert obj["bound"] == "alu" and obj["visits"] == (1 << 40) + (1 << 39)
    assert abs(obj["frac"] - ((1 << 39) + (1 << 39)) / 0.02 / bench.PEAK_INT32_LANE_OPS) < 1e-12
