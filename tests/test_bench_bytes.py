"""Bytes that bench.py holds a launch of each smoothing class to, and the length of its line (no GPU)."""
import json

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


def test_line_stays_short():
    """A line of every variant fits in 6 KB: per variant at most 330 characters."""
    dev = dict(phi_rel_per_level=[1.23456789012e-11] * 16, force_rel_per_level=[1.23456789012e-11] * 16, phi_rel=1.23456789012e-11,
               force_rel=3.45678901234e-11)
    r = dict(ms_per_solve=1234.567, wall_ms_per_step=1234.567, cycles_per_level=[18] * 5, outer_steps_per_level=[6] * 5,
             linf_force_error=1.0078651234567, deviation_from_fp64=dev, kernels={str(k): dict(launches=1) for k in range(100)})
    line = bench.variant_line(r)
    assert len(json.dumps(line)) <= 330
    assert line["deviation_from_fp64"] == dict(phi_rel=1.23457e-11, force_rel=3.45679e-11)
    assert bench.variant_line(dict(r, deviation_from_fp64=None))["deviation_from_fp64"] is None
