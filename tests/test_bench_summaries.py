"""The profile summaries of the benchmark: a kernel kind made of several kernels (the stage
updates of the z sweep) counts with all its dispatches, for bytes, times and shader counters."""
import csv
import os

import pytest

bench = pytest.importorskip("bench")

Z = [f"void cns::k_sweep<double, 2, {m}, false, 0>(cns::Launch)" for m in (2, 3, 4)]
Y = "void cns::k_sweep<double, 1, 1, false, 0>(cns::Launch)"


def test_kind_totals_are_means_over_every_dispatch():
    fetch = {Z[0]: [10.0], Z[1]: [16.0, 16.0], Z[2]: [22.0], Y: [11.0] * 4}
    write = {Z[0]: [5.0], Z[1]: [8.0, 8.0], Z[2]: [5.0], Y: [5.0] * 4}
    # the trace takes three steps
    dur = {Z[0]: [400] * 3, Z[1]: [500] * 6, Z[2]: [540] * 3, Y: [300] * 12}
    z = bench.kind_totals(fetch, write, dur)["sweep_z_rk4"]
    assert z == {"bytes_per_launch": 22, "fetch_bytes": 16, "write_bytes": 6, "avg_launch_ns": 485.0, "dispatches": 4}
    assert bench.kind_totals(fetch, write, dur)["sweep_y"]["bytes_per_launch"] == 16


def test_shader_counters_take_the_time_of_the_whole_kind(tmp_path):
    os.makedirs(tmp_path / "sq1")
    with open(tmp_path / "sq1" / "x_counter_collection.csv", "w", newline="") as f:
        w = csv.DictWriter(f, ["Kernel_Name", "Counter_Name", "Counter_Value"])
        w.writeheader()
        for name, v in ((Z[0], 7.0), (Z[1], 8.0), (Z[1], 8.0), (Z[2], 9.0)):
            w.writerow({"Kernel_Name": name, "Counter_Name": "SQ_INSTS_VALU", "Counter_Value": v})
    for order in (Z, Z[::-1]):
        got = bench.summarize_sq(str(tmp_path), 8, {k: t for k, t in zip(order, ([400], [500, 500], [540]))})
        assert got["sweep_z_rk4"] == {"SQ_INSTS_VALU": 8.0, "_avg_ns": 485.0}
