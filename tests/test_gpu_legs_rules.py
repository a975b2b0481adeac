"""Streamed legs of coarse levels (np_stream.hip, boundary rule) against the per-pass kernels, bit for bit, where
their ghost values differ by axis: the last point at an even or an odd index, x_N = 1 or a coefficient.

Coarse levels of more than 1024 blocks of 8 x 8 x 8 points are streamed.  A first coarse level has N = N^0 / 2 and
coefficient -1 on every axis; a second one x_N = 1 where N^0 = 2 mod 4 and -1 elsewhere; a third one -1/3, x_N = 1 or
-3 where N^0 = 2, 4 or 6 mod 8.
"""
import pytest
import torch

from paper_2001_02327_amd import workloads as W
from paper_2001_02327_amd.solver import NestedPoissonSolver

pytestmark = pytest.mark.gpu

KW = [dict(), dict(n_pre=1, n_post=2), dict(precision="fp32_dc", inner_cycles=2),
      dict(precision="fp32_dc", inner_cycles=2, n_pre=1, coarse_post=2)]


def _solve(g, rho, po, kw):
    s = NestedPoissonSolver(g, max_cycles=6, **kw)
    st = s.solve(rho, po, allow_notconv=True)
    out = [s.potential(0)] + list(s.forces(0)), s.history(0), list(st["cycles"])
    torch.cuda.synchronize()
    s.close()
    return out


def _same(n, kw):
    g = W.Geometry(dim=3, n=[tuple(n)], off=[(0, 0, 0)], lo0=(0.0, 0.0, 0.0), dx0=1.0 / 32)
    rho, po = W.make_inputs(g, W.Plummer([(1.0, 0.3, tuple(0.4 * a / 32 for a in n))]), device="cuda")
    a, b = _solve(g, rho, po, kw), _solve(g, rho, po, dict(kw, sweep="half"))
    assert a[1:] == b[1:]
    for x, y in zip(a[0], b[0]):
        assert bool(torch.isfinite(x).all()) and torch.equal(x, y)


def _rotations(n):
    return [n, n[1:] + n[:1], n[2:] + n[:2]]


_ids = dict(ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "-".join("%s=%s" % a for a in v.items()) or "fp64")


# first coarse level 102 x 86 x 92 (all even), 102 x 87 x 91 (one axis even)
@pytest.mark.parametrize("n", _rotations((202, 170, 182)) + _rotations((202, 172, 180)), **_ids)
@pytest.mark.parametrize("kw", KW, **_ids)
def test_first_level(n, kw):
    _same(n, kw)


# second one 84 x 87 x 88: x_N = 1, -1, -1 (the first one 167 x 174 x 176)
@pytest.mark.parametrize("n", _rotations((332, 346, 350)), **_ids)
@pytest.mark.parametrize("kw", KW, **_ids)
def test_second_level(n, kw):
    _same(n, kw)


# third one 2 x 256 x 257: -3, -1/3, x_N = 1 (the second one 4 x 513 x 513: x_N = 1, x_N = 1, -1)
@pytest.mark.parametrize("n", _rotations((12, 2048, 2050)), **_ids)
@pytest.mark.parametrize("kw", KW, **_ids)
def test_third_level(n, kw):
    _same(n, kw)


# mixed precisions with level 0 per pass: streamed from a first coarse level of 2^23 points on (208 x 206 x 202)
@pytest.mark.parametrize("kw", [dict(precision="fp16s_dc", inner_cycles=2), dict(precision="fp32_dc", n_pre=1, n_post=2)], **_ids)
def test_first_level_mixed(kw):
    _same((414, 410, 402), kw)
