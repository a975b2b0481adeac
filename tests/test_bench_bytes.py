"""Bytes that bench.py holds a launch of each smoothing class to (no GPU)."""
import pytest

from conftest import ROOT  # noqa: F401  (the repository's root on sys.path)

import bench


def test_per_pass_classes():
    assert bench.smoothing_elements(2, 1, False, 60, 20) == dict(smooth=1.5, seeded=2.0, full=2.5, full_res=3.0)
    assert bench.smoothing_elements(8, 3, False, 60, 0)["seeded"] == 1.5


def test_fp64_legs():
    # no leg starts from zero, whatever the outer steps of other variants were
    assert bench.smoothing_elements(8, 2, True, 62, 0) == dict(smooth=2.375, full=2.125, full_res=2.625)


@pytest.mark.parametrize("cycles,outer,smooth", [(62, 62, 2.125), (62, 31, 2.25), (18, 5, (17 * 2.125 + 1.625 - 4 * 0.5) / 36 + 1.3125)])
def test_fp32_legs(cycles, outer, smooth):
    """The mean over a step's down legs, the first of which starts from zero (1.625), and its up legs (2.625)."""
    assert bench.smoothing_elements(4, 2, True, cycles, outer)["smooth"] == pytest.approx(smooth, rel=1e-12)
