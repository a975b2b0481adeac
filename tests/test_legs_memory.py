"""A handle without the memory for the buffers of the fused V-cycle legs (no GPU: the stand-in for the
runtime has a limit): it is created all the same and runs the per-pass kernels, and only what those
need may fail it."""
import json

import pytest

from hip_stub import run

# a batch of eight patches (3-D, 2-D: four), a stack, the mixed precisions' coarse legs
CASES = {
    "batch3d": ("geom([(64,) * 3] + [(16,) * 3] * 8, [(0, 0, 0)] + [(12 + 32 * (c & 1), 12 + 32 * (c >> 1 & 1), 12 + 32 * (c >> 2)) for c in range(8)], [-1] + [0] * 8)", {}),
    "stack3d": ("geom([(32, 32, 32), (40, 28, 30)], [(0, 0, 0), (4, 6, 8)])", {}),
    "one2d": ("geom([(126, 128)])", {}),
    "fp32": ("geom([(64, 64, 64)])", dict(precision="fp32_dc")),
    "fp16": ("geom([(128, 128, 128)])", dict(precision="fp16s_dc", n_pre=1, coarse_post=2)),
}

CODE = r"""
import json
g, kw = %s, %r
def go(limit, **more):
    S.stub_limit(limit)
    h = create(g, **dict(kw, **more))
    used = S.stub_used()
    S.stub_clear()
    if not isinstance(h, ctypes.c_void_p):
        return h, 0, [], L.nested_poisson_last_error(None).decode(), S.stub_live()
    rc, ks, err = solve(h, g), [k.split("(")[0] for k in kernels()], L.nested_poisson_last_error(h).decode()
    L.nested_poisson_destroy(h)
    return rc, used, ks, err, S.stub_live()
full, half = go(-1), go(-1, sweep="half")
short = go(full[1] - 1)
print(json.dumps([full, half, short, go(short[1]), go(short[1] - 1)]))
"""


@pytest.mark.parametrize("case", CASES)
def test_legs_are_optional(case):
    g, kw = CASES[case]
    full, half, short, exact, none = json.loads(run(CODE % (g, kw)))
    legs = ("k_tile", "k_leg3")
    assert full[0] == half[0] == 0 and any(x in k for k in full[2] for x in legs)
    # one byte short of the legs' buffers: no legs, the launches of the per-pass cycle
    assert short[0] == 0 and short[3] == "" and short[1] < full[1]
    assert short[2] == half[2] and not any(x in k for k in short[2] for x in legs)
    assert exact[:3] == short[:3]
    # what the per-pass cycle needs is required
    assert none[0] == -2 and "hipMalloc" in none[3]
    assert [r[4] for r in (full, half, short, exact, none)] == [0] * 5
