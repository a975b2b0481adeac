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
