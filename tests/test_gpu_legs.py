"""Fused V-cycle legs (the default sweep mode, one or two pre- and post-smoothing
sweeps) against the per-pass kernels (sweep="half").

One launch takes a multigrid level down or up.  3-D: blocks of the level in LDS
on levels of at most 1024 blocks of 8 x 8 x 8 points (batch members included),
columns streamed through it on the larger ones; FP64 and FP32 every level, FP16
storage the coarse levels that fit the block form.  2-D: blocks of 16^2 points, of 32^2 for the leg
with the norm where the small ones are more than 512; in the mixed precisions the
coarse levels.  Every operation and its order are those of
the per-pass kernels, so potentials, forces, cycle counts and residual histories
are compared for equality, bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2001_02327_amd import workloads as W
from paper_2001_02327_amd.solver import NestedPoissonSolver

pytestmark = pytest.mark.gpu


def _solve(wl, **kw):
    rho, po = W.make_inputs(wl.geom, wl.prob, device="cuda")
    s = NestedPoissonSolver(wl.geom, **kw)
    st = s.solve(rho, po, allow_notconv=True)
    out = [s.potential(l) for l in range(wl.geom.nlevels)]
    for l in range(wl.geom.nlevels):
        out += list(s.forces(l))
    out = [a.cpu().numpy() for a in out]
    hist = [s.history(l) for l in range(wl.geom.nlevels)]
    s.close()
    return out, hist, list(st["cycles"])


def _same(wl, **kw):
    a, b = _solve(wl, **kw), _solve(wl, sweep="half", **kw)
    assert a[2] == b[2] and a[1] == b[1]
    for x, y in zip(a[0], b[0]):
        assert np.isfinite(x).all()
        assert np.array_equal(x, y)


def _one(*n):
    g = W.Geometry(dim=3, n=[tuple(n)], off=[(0, 0, 0)], lo0=(0.0, 0.0, 0.0), dx0=1.0 / 32)
    return W.Workload("one%s" % (n,), g, W.Plummer([(1.0, 0.3, tuple(0.4 * a / 32 for a in n))]))


# single levels: a column and block exactly filled, one point more and one less in
# each direction; flat and long ones; both sides of the limit between the forms
SIZES = [(8, 8, 8), (10, 8, 14), (16, 18, 20), (40, 38, 36), (72, 68, 34), (80, 80, 80), (88, 88, 72), (108, 102, 90),
         (110, 104, 92), (106, 100, 110), (120, 114, 80), (122, 116, 82), (118, 112, 78), (200, 200, 12), (24, 200, 180),
         (40, 44, 400)]


@pytest.mark.parametrize("n", SIZES, ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("pre,post", [(2, 1), (1, 2)])
def test_sizes_fp64(n, pre, post):
    _same(_one(*n), n_pre=pre, n_post=post, max_cycles=8)


# both sides of the limits between the block shapes (256 blocks), on level 0 (24 | 26, 40 | 42,
# 48 | 52 points an axis) and on the first coarse level (24 | 26, 38 | 41)
@pytest.mark.parametrize("n", [22, 24, 38, 40, 46, 50, 74, 80])
@pytest.mark.parametrize("kw", [dict(n_pre=2, n_post=1), dict(n_pre=1, n_post=2), dict(precision="fp32_dc", inner_cycles=2),
                                dict(precision="fp32_dc", n_pre=1, inner_cycles=2, coarse_post=2)],
                         ids=lambda kw: "-".join("%s=%s" % a for a in kw.items()))
def test_block_shapes(n, kw):
    _same(_one(n, n, n), max_cycles=8, **kw)


# the coarse levels' boundary rules in block form, on each axis in turn: last point x_N = 1 with N
# odd (51) and even (22, 28) on the second level, below it a coefficient of -3 with N odd (11) and
# even (14)
@pytest.mark.parametrize("n", [(200, 84, 108), (84, 108, 200), (108, 200, 84)], ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("kw", [dict(n_pre=2, n_post=1), dict(n_pre=1, n_post=2),
                                dict(precision="fp32_dc", inner_cycles=2), dict(precision="fp16s_dc", inner_cycles=2, n_pre=1, coarse_post=2)],
                         ids=lambda kw: "-".join("%s=%s" % a for a in kw.items()))
def test_boundary_rules(n, kw):
    _same(_one(*n), max_cycles=8, **kw)


@pytest.mark.parametrize("kw", [dict(), dict(n_pre=1), dict(n_post=2), dict(n_pre=1, coarse_post=2),
                                dict(buffer="interp"), dict(stop_rule="force_delta")],
                         ids=lambda kw: "-".join("%s=%s" % a for a in kw.items()) or "default")
@pytest.mark.parametrize("wl", [W.c2_plummer(16), W.c3_plummer_offset(96), W.box_plummer_3d(4)], ids=lambda w: w.name)
def test_nested_fp64(wl, kw):
    _same(wl, **kw)


@pytest.mark.parametrize("n", [16, 32, 64])
def test_batches(n):
    # members side by side in one launch: the block form for 16, streamed columns for 64
    _same(W.many_patches_3d(n, 2, 8, depth2=True))


@pytest.mark.parametrize("precision", ["fp32_dc", "fp16s_dc"])
@pytest.mark.parametrize("kw", [dict(), dict(n_pre=1, coarse_post=2), dict(n_pre=1, n_post=2)],
                         ids=lambda kw: "-".join("%s=%s" % a for a in kw.items()) or "default")
@pytest.mark.parametrize("wl", [W.c2_plummer(32), W.c2_plummer(132, 1), W.box_plummer_3d(4)], ids=lambda w: w.name)
def test_mixed(wl, kw, precision):
    _same(wl, precision=precision, inner_cycles="adaptive", **kw)


# 2-D: blocks exactly filled and one point more, several blocks, both block sizes
SIZES2 = [(8, 8), (16, 16), (30, 14), (32, 34), (62, 62), (126, 128), (254, 62), (128, 510), (510, 512), (1022, 1024)]


@pytest.mark.parametrize("n", SIZES2, ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("pre,post", [(2, 1), (1, 2)])
def test_sizes_2d(n, pre, post):
    g = W.Geometry(dim=2, n=[n], off=[(0, 0, 0)], lo0=(0.0, 0.0, 0.0), dx0=1.0 / 32)
    _same(W.Workload("one%s" % (n,), g, W.Gaussian(0.15, 1.0)), n_pre=pre, n_post=post, max_cycles=8)


@pytest.mark.parametrize("kw", [dict(), dict(n_pre=1, coarse_post=2), dict(buffer="interp"), dict(stop_rule="force_delta"),
                                dict(precision="fp32_dc", inner_cycles=2),
                                dict(precision="fp16s_dc", inner_cycles="adaptive", n_pre=1, coarse_post=2)],
                         ids=lambda kw: "-".join("%s=%s" % a for a in kw.items()) or "default")
@pytest.mark.parametrize("wl", [W.c1_gaussian_2d(64), W.paper2d(256), W.box_gaussian_2d(2)], ids=lambda w: w.name)
def test_nested_2d(wl, kw):
    _same(wl, **kw)


def test_large():
    # 260^3: streamed legs on the three largest levels, blocks below
    _same(W.c2_plummer(260, 1))


def test_norms_after_a_failed_solve():
    """A solve that ends early (non-finite density) leaves nothing behind in the norms of the
    handle's next one."""
    wl = W.c2_plummer(32)
    rho, po = W.make_inputs(wl.geom, wl.prob, device="cuda")
    ref, hist, cycles = _solve(wl)
    s = NestedPoissonSolver(wl.geom)
    bad = [r.clone() for r in rho]
    bad[1][3, 4, 5] = float("nan")
    with pytest.raises(Exception):
        s.solve(bad, po)
    st = s.solve(rho, po)
    assert list(st["cycles"]) == cycles
    assert [s.history(l) for l in range(wl.geom.nlevels)] == hist
    for l in range(wl.geom.nlevels):
        assert np.array_equal(s.potential(l).cpu().numpy(), ref[l])
    s.close()


@pytest.mark.parametrize("n", [(8, 8, 8), (10, 8, 14), (16, 18, 20), (54, 22, 30), (58, 28, 40), (110, 46, 62), (120, 54, 34),
                               (24, 100, 90), (200, 200, 12), (260, 260, 260)], ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("pre,cycles", [(2, 2), (1, "adaptive")])
def test_sizes_fp32(n, pre, cycles):
    # multigrid level 0 streamed at every size, from zero and from the previous cycle
    _same(_one(*n), precision="fp32_dc", n_pre=pre, inner_cycles=cycles, max_cycles=12)


def test_largest_coarse_levels():
    # a first coarse level of 2^23 points and more: streamed in FP32 under FP16 storage too
    _same(W.c2_plummer(512, 1), precision="fp16s_dc", inner_cycles="adaptive", n_pre=1, coarse_post=2, max_cycles=6)
