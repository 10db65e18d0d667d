"""The headline leg's figures are not made from the rows it steps over: its
planner looks up a few records of a row's index."""
import bench


def test_range_leg_counts_no_row_bytes():
    leg = dict(kms=8.0, launches=10, steps=2_000_000, pairs=10, entries=0)
    a, b = bench._latency(leg, "range_query"), bench._latency(dict(leg, entries=10 ** 12), "range_query")
    assert a == b and a["bound"] == "latency" and a["steps_per_us"] == 250.0
    if a["traffic"] is None:                             # other sources than the counters were taken on
        assert a["achieved"] is None and a["frac"] is None
    else:
        assert abs(a["achieved"] - a["traffic"] / 0.8e-3 / 1e9) < 1e-6 * a["achieved"]
