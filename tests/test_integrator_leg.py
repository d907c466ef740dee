"""The benchmark's integrator comparison runs from one slice on: a single drift-kick
slice takes every particle beyond the rings' 0.05 m aperture, so the leg has its own.
"""

import pytest

from workloads import Beam

pytestmark = pytest.mark.gpu


def test_every_method_has_a_row_for_each_slice_count():
    import bench
    table = bench.integrator_leg(Beam(), n=64, slices=(1, 8))["one_turn"]
    for style, rows in table.items():
        want = [N for N in (1, 8) if "_romberg" not in style or N >= 2 ** (int(style[-1]) - 1)]
        assert [r["slices"] for r in rows] == want, style
    err = {N: r["orbit_err_over_sigma"] for N, r in zip((1, 8), table["dk_kick"])}
    assert err[8] < 0.1 * err[1]         # second order: 1/64
