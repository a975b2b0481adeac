"""Which kernel a convolution of the guess network goes to (no GPU: the launches are logged by the
stand-in for the runtime)."""
import pytest

from hip_stub import run


def _kernel(call):
    """Signature of the convolution kernel that `call` launches."""
    out = run("rc = L.%s\nassert rc == 0, rc\nfor k in kernels(): print(k)\n" % call)
    return [k for k in out.splitlines() if "conv" in k][0]


@pytest.mark.parametrize("cin,cout", [(2, 16), (16, 16), (16, 1)])
def test_rows_of_a_buffer(cin, cout):
    """A row of the inference layers is one buffer of less than 2^31 bytes; longer rows take the general kernel."""
    call = "np_net_conv3d_fwd_mfma(64, %d, 64, 64, %d, 0, 1, 1, 1, %%d, 64, None)" % (cin, cout)
    assert "k_conv_mfma" in _kernel(call % ((1 << 26) - 1))
    assert "k_conv_fwd_t" in _kernel(call % (1 << 26))
    assert "k_conv_fwd_t" in _kernel(call % ((1 << 26) + 40))


def _planes(Z, cols, slots):
    """Planes per workgroup by trying every number of ranges."""
    best = None
    for n in range(1, Z + 1):
        k = -(-Z // n)
        cost = -(-(cols * -(-Z // k)) // slots) * (k + 2)
        if best is None or cost < best[0]:
            best = (cost, k)
    return best[1]


def test_planes_per_workgroup():
    """The inference layers' ranges of planes: the cheapest of all, found without trying every one."""
    shapes = [(1, z, y, x) for z in (1, 2, 3, 17, 64, 258, 1000, 4000) for y, x in ((1, 1), (9, 40), (130, 130))] + [(7, 300, 66, 66)]
    code = r"""
import time
for B, Z, Y, X in %r:
    S.stub_clear()
    assert L.np_net_conv3d_fwd_mfma(64, 2, 64, 64, 16, 0, B, Z, Y, X, 64, None) == 0
    print(S.stub_log().split()[1].decode())
t = time.perf_counter()
assert L.np_net_conv3d_fwd_mfma(64, 2, 64, 64, 16, 0, 1, 1 << 30, 1, 1, 64, None) == 0
print(time.perf_counter() - t)
""" % shapes
    *grids, seconds = run(code).split()
    for (B, Z, Y, X), g in zip(shapes, grids):
        cols = B * -(-X // 16) * -(-Y // 8)  # two rows per wavefront, four wavefronts
        assert int(g) == cols * -(-Z // _planes(Z, cols, 4 * 256)), (B, Z, Y, X)
    assert float(seconds) < 0.25  # (2^30 ranges take seconds)
