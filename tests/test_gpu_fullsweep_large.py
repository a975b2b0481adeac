"""Full sweeps where the default schedule chooses them: three or more sweeps on level grids whose full sweep starts
at least 4096 wavefronts (one or two sweeps run fused legs, and smaller grids half sweeps).  The next cycle's first
pre-smoothing sweep, which completes the stop test's norm, is taken over (or dropped when the level stops).  Against the
half sweeps, bit for bit.
"""
import pytest
import torch

from paper_2001_02327_amd import workloads as W
from paper_2001_02327_amd.solver import NestedPoissonSolver

pytestmark = pytest.mark.gpu


def _solve(wl, rho, po, **kw):
    s = NestedPoissonSolver(wl.geom, **kw)
    s.set_profiling(True)
    st = s.solve(rho, po, allow_notconv=True)
    prof = {k: c for k, (c, _) in s.profile().items()}
    out = [s.potential(0)] + list(s.forces(0))
    hist = s.history(0)
    torch.cuda.synchronize()
    s.close()
    return out, hist, list(st["cycles"]), prof


@pytest.mark.parametrize("pre,post,cycles", [(3, 1, 50), (1, 3, 50), (3, 2, 4)])
def test_full_sweeps_of_a_large_level(pre, post, cycles):
    wl = W.c5_two_plummer(N=512, nlevels=1)
    rho, po = W.make_inputs(wl.geom, wl.prob, device="cuda")
    a = _solve(wl, rho, po, n_pre=pre, n_post=post, max_cycles=cycles)
    b = _solve(wl, rho, po, n_pre=pre, n_post=post, max_cycles=cycles, sweep="half")
    n = a[2][0]
    # every sweep of every cycle, the first one of all but the first cycle as the norm pass before it
    assert a[3]["full"] == n * (pre + post) - (n - 1) and a[3]["full_res"] == n and a[3]["smooth"] == 0
    assert b[3]["full"] == b[3]["full_res"] == 0 and b[3]["smooth"] == 2 * n * (pre + post)
    assert a[3]["restrict"] == b[3]["restrict"] == n
    assert a[1:3] == b[1:3]
    for x, y in zip(a[0], b[0]):
        assert torch.equal(x, y)


def test_legs_with_one_or_two_sweeps():
    wl = W.c5_two_plummer(N=512, nlevels=1)
    rho, po = W.make_inputs(wl.geom, wl.prob, device="cuda")
    a = _solve(wl, rho, po)
    assert a[3]["full"] == a[3]["full_res"] == a[2][0] and a[3]["restrict"] == a[3]["prolong"] == a[3]["smooth"] == 0
