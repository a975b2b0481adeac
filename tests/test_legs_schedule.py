"""Which kernels run multigrid level 0 in the default schedule and beside it (no GPU: the launches are logged by the
stand-in for the runtime).  Profiling classes cannot tell fused legs from full or half sweeps, whose classes they share."""
import pytest

from hip_stub import run

SCHEDULES = [
    # (cells, settings) -> kernels of multigrid level 0's sweeps and whether the residual's restriction is a launch
    ((512, 512, 512), dict(), "k_leg3", False),
    ((512, 512, 64), dict(), "k_leg3", False),
    ((64, 64, 64), dict(), "k_tile_down3", False),
    ((512, 512, 512), dict(n_pre=3), "k_full_sweep3", True),
    ((512, 512, 512), dict(n_post=3), "k_full_sweep3", True),
    ((512, 512, 64), dict(n_pre=3), "k_smooth", True),
    ((256, 256, 256), dict(n_pre=3), "k_smooth", True),
    ((512, 512, 512), dict(sweep="half"), "k_smooth", True),
    ((64, 64, 64), dict(sweep="full_all"), "k_full_sweep3", True),
    ((64, 64, 64), dict(precision="fp32_dc"), "k_leg3<float", False),
    ((64, 64, 64), dict(precision="fp32_dc", n_post=2), "k_smooth", True),
    ((62, 64, 64), dict(precision="fp32_dc"), "k_smooth", True),
    ((64, 64, 64), dict(precision="fp16s_dc"), "k_smooth", True),
]


@pytest.mark.parametrize("n,kw,kernel,restricts", SCHEDULES)
def test_schedule_of_a_level(n, kw, kernel, restricts):
    """What runs on multigrid level 0: fused legs with one or two sweeps, full sweeps on large grids with more,
    half sweeps on smaller ones; in the mixed precisions legs with FP32 storage, one post-smoothing sweep and an even
    row length.  The full sweeps' norm pass is the next cycle's first sweep: one more of them than the cycles hold."""
    out = run(r"""
g = geom([%r])
h = create(g, **%r)
S.stub_clear()
assert solve(h, g, 3) == 0
for k in kernels(): print(k.replace("void ", "", 1).split("(")[0])
""" % (n, kw)).splitlines()
    forms = ("k_leg3", "k_tile_down3", "k_full_sweep3", "k_smooth")
    first = [k for k in out if k.startswith(forms)][0]
    assert first.startswith(kernel), out
    assert any(k.startswith(("k_restrict", "k_resid_restrict", "k_black_restrict")) for k in out) == restricts
    fulls = sum(k.startswith("k_full_sweep3") for k in out)
    if kernel == "k_full_sweep3":
        sweeps = kw.get("n_pre", 2) + kw.get("n_post", 1)
        assert fulls == 3 * sweeps + 1  # the first sweep of cycles 2 and 3 and a dropped one end the norms
    else:
        assert fulls == 0
