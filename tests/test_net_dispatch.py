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


@pytest.mark.parametrize("cin,cout,small,large", [
    (16, 1, [(1, 18, 18, 18), (1, 50, 50, 50), (4, 34, 34, 34), (1, 130, 130, 6), (1, 258, 258, 6), (1, 4000, 3, 3)],
     [(1, 58, 58, 58), (1, 66, 66, 66), (1, 130, 130, 130), (1, 130, 130, 34), (1, 6, 258, 258)]),
    (2, 16, [(1, 130, 130, 6), (1, 130, 130, 17), (1, 258, 258, 17), (16, 18, 18, 18)],
     [(1, 1, 1, 1), (1, 18, 18, 18), (1, 130, 130, 14), (1, 130, 130, 130), (1, 6, 130, 130)]),
    (16, 16, [(1, 130, 130, 3), (1, 130, 130, 6), (1, 4000, 3, 3)],
     [(1, 1, 1, 1), (1, 18, 18, 18), (1, 130, 130, 10), (1, 3, 130, 130), (1, 130, 130, 130)])])
def test_training_forward(cin, cout, small, large):
    """The forward pass of a training layer: a thread per voxel on volumes that fill their blocks badly (or, with
    one output channel, are small), blocks on the others; the rounded pass in blocks always."""
    call = "np_net_conv3d_fwd(64, %d, 64, 64, %d, 1, %%d, %%d, %%d, %%d, 64, None)" % (cin, cout)
    blocks = {(16, 1): "k_conv16_to_few", (2, 16): "k_conv_few_to16", (16, 16): "k_conv16_mfma"}[cin, cout]
    for s in small:
        assert "k_conv_fwd_t<%d, %d, float, float>" % (cin, cout) in _kernel(call % s), s
    for s in large:
        assert blocks in _kernel(call % s), s
    for s in small + large:
        assert blocks in _kernel(call.replace("fwd(", "fwd_round(").replace(", 1, %d", ", %d", 1) % s), s


def test_data_gradient():
    call = "np_net_conv3d_bwd_data(64, 16, 64, 2, %d, %d, %d, %d, 64, None)"
    for s in [(1, 4000, 3, 3), (1, 40000, 3, 3), (4, 1000, 4, 5)]:
        assert "k_conv_bwd_data" in _kernel(call % s), s
    for s in [(1, 1, 1, 1), (1, 1000, 3, 3), (1, 130, 130, 3), (1, 4000, 6, 6), (1, 130, 130, 130)]:
        assert "k_conv16_to_few_f32<2, true>" in _kernel(call % s), s
