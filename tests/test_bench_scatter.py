"""What bench.py reports of the feature scatter (no GPU needed)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench


def test_no_rate_over_the_time_of_two_kernels():
    """Where some levels have a launch of their own, the scatter's time covers
    requests that are not counted: the count alone, no rate. Elsewhere the
    step's requests over the step's scatter time, in any number of launches."""
    scatter = {"ms_per_launch": 0.25, "launches_per_step": 4.0, "ms_per_step": 1.0}
    got = bench.atomic_rate(scatter, 14_000_000, {2, 0})
    assert got == {"atomic_requests": 14_000_000, "merged_levels": [0, 2]}
    got = bench.atomic_rate(scatter, 14_000_000, set())
    assert got["atomic_Greq_s"] == 14.0
    assert got["frac_of_atomic_ceiling"] == pytest.approx(14.0 / bench.ATOMIC_GREQ_S, abs=1e-4)


@pytest.mark.parametrize("compute_units,want", [(256, {0, 1, 2}), (1024, {0, 1})])
def test_merged_levels_follow_the_device(compute_units, want):
    """A workgroup takes the batch's share of a compute unit, 4096 to 16384
    points, and needs two per footprint of a node: 1089 footprints on maps of
    32 x 32 texels, 4225 on 64 x 64. Over all nodes of a level the batch does."""
    cfg = type("Maps", (), {"res": (32, 32, 64, 64)})
    nodes, paired = [1, 8, 1, 5000], {0, 1, 2, 3}
    assert bench.merged_levels(cfg, nodes, paired, 1 << 20, compute_units) == want
    assert bench.merged_levels(cfg, nodes, paired, (1 << 17) - 1, compute_units) == set()
