"""How the host waits for a stop test's norm (no GPU: the stand-in for the runtime lets the norm out only
when the stream is synchronised, or has been queried often enough): by polling pinned memory, or by the
stream's own wait where the device's scheduling flags ask for a core to be left free."""
import json

import pytest

from hip_stub import run

CODE = r"""
import json
g = geom(%s)
S.stub_flags(%d)
S.stub_defer(3)
h = create(g, **%r)
S.stub_clear()
rc = solve(h, g)
print(json.dumps([rc, S.stub_syncs(), S.stub_queries(), sum("k_publish" in k for k in kernels())]))
"""

ONE, BATCH = "[(16, 16, 16)]", "[(32,) * 3] + [(8,) * 3] * 2, [(0, 0, 0), (2, 4, 4), (20, 4, 4)], [-1, 0, 0]"


@pytest.mark.parametrize("geom", [ONE, BATCH], ids=["one", "batch"])
@pytest.mark.parametrize("kw", [{}, dict(sweep="half"), dict(precision="fp32_dc"), dict(stop_rule="force_delta")],
                         ids=lambda kw: "-".join(kw.values()) or "fp64")
def test_wait_follows_the_scheduling_flags(geom, kw):
    for flags in (2, 4):  # hipDeviceScheduleYield, hipDeviceScheduleBlockingSync
        rc, syncs, queries, reads = json.loads(run(CODE % (geom, flags, kw)))
        assert rc == 0 and syncs == reads > 0 and queries == 0
    for flags in (0, 1, 8):  # automatic, hipDeviceScheduleSpin, a flag of another kind
        rc, syncs, queries, reads = json.loads(run(CODE % (geom, flags, kw)))
        assert rc == 0 and syncs == 0 and queries >= 3 * reads > 0
