"""The coarse tail (one workgroup takes the smallest multigrid levels down and up,
a slot of a level per thread, several with the per-pass kernels above it)
against the CPU oracle after a pinned number of cycles, at the FP64 bars of the
parity tests (1e-12 of max |Phi|, 1e-11 of max |F|): levels of one wavefront and of
several, around 64 and 1024 slots, thin ones, both dimensions.
"""
import numpy as np
import pytest
import torch

from oracle import core
from paper_2001_02327_amd import workloads as W
from paper_2001_02327_amd.solver import NestedPoissonSolver

pytestmark = pytest.mark.gpu

SIZES = [(4, 4, 4), (8, 8, 8), (10, 8, 14), (14, 16, 18), (20, 22, 24), (24, 24, 24), (26, 24, 24), (32, 32, 32), (30, 60, 6),
         (6, 6, 60), (8, 8), (20, 22), (30, 32), (62, 62), (64, 64), (90, 90), (30, 100), (128, 24)]


@pytest.mark.parametrize("sweep", ["full", "half"])
@pytest.mark.parametrize("n", SIZES, ids=lambda n: "x".join(map(str, n)))
def test_tail_against_oracle(n, sweep):
    d = len(n)
    g = W.Geometry(dim=d, n=[n], off=[(0, 0, 0)], lo0=(0.0, 0.0, 0.0), dx0=1.0 / 32)
    prob = (W.Plummer([(1.0, 0.3, tuple(0.4 * a / 32 for a in n))]) if d == 3 else W.Gaussian(0.15, 1.0))
    wl = W.Workload("tail", g, prob)
    rho, po = W.make_inputs(g, wl.prob, device="cuda")
    s = NestedPoissonSolver(g, sweep=sweep)
    s.set_fixed_cycles([3])
    s.solve(rho, po, allow_notconv=True)
    phi = s.potential(0).cpu().numpy()
    F = [a.cpu().numpy() for a in s.forces(0)]
    s.close()
    rho, po = W.make_inputs(g, wl.prob, device="cpu")
    ref = core.solve(g, [r.numpy() for r in rho], po.numpy(), fixed_cycles=[3])["phi"][0]
    Fo = core.forces(d, g.dx(0), ref)
    assert np.abs(phi - ref).max() <= 1e-12 * np.abs(ref).max()
    fmax = max(np.abs(x).max() for x in Fo)
    for a, b in zip(F, Fo):
        assert np.abs(a - b).max() <= 1e-11 * fmax
