"""The counter traffic that bench.py reports was taken from the kernels as they
are: each entry's digest is that of its sources."""
import pytest

import bench


@pytest.mark.parametrize("stage", sorted(bench.MEASURED_TRAFFIC))
def test_counters_belong_to_the_sources(stage):
    _, _, read, written = bench.MEASURED_TRAFFIC[stage]
    assert bench.measured_traffic(stage) == read + written
