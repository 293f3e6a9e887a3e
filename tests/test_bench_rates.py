"""The marchers' benchmark rows divide no count of one launch by another's time."""
import inspect

import bench_workloads


def test_marcher_rows_hold_no_rate_of_two_launches():
    # the timed launch skips samples that the counting launch visits
    for workload in (bench_workloads.iso, bench_workloads.ea):
        source = inspect.getsource(workload)
        assert "sample_count() / ms" not in source and "taken" not in source
        assert "_per_s" not in source and "gbs" not in source
