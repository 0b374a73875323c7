"""What bench.py reports beside its timings, without a GPU."""

import bench
import paper_2510_16045_amd as ams


def test_traffic_is_reported_for_the_kernel_that_was_profiled_only():
    column = bench.measured_traffic(ams, "gate_up", "fp5.33-e2m3", 1, "column_kernel")
    assert column == 79206371 + 57344
    assert bench.measured_traffic(ams, "gate_up", "fp5.33-e2m3", 1, "multi_kernel") is None
    assert bench.measured_traffic(ams, "gate_up", "fp5.33-e2m3", 1, "slice_kernel") == 79165645 + 57344
    assert bench.measured_traffic(ams, "gate_up", "fp5.33-e2m3", 2, "column_kernel") is None
