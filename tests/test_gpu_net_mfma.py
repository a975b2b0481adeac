"""The inference layers on the matrix cores at the edges of their blocks (16 voxels
along x, 2 or 4 rows per wavefront, ranges of planes) against FP64 convolutions of
the same bfloat16 inputs and weights.

Tolerance: 27 cin products and the bias are summed in FP32, each addition within
2^-24 of the sum of the magnitudes S, so within 433 x 2^-24 S; a bfloat16 output adds half
a unit in the last place, 2^-9 of the value (2^-8 with the rounding of the sum).
"""
import ctypes

import pytest
import torch

from paper_2001_02327_amd import _lib

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1, 1), (1, 2, 3, 5), (1, 3, 8, 15), (2, 4, 9, 16), (1, 5, 7, 17), (1, 6, 16, 18), (1, 18, 17, 19),
          (1, 20, 33, 34), (2, 7, 40, 49), (4, 300, 18, 17), (1, 1030, 16, 64)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("cin,cout", [(2, 16), (16, 16), (16, 1)])
def test_layer(cin, cout, shape):
    B, Z, Y, X = shape
    gen = torch.Generator().manual_seed(1000 * cin + X)
    x = torch.randn(B, Z, Y, X, cin, generator=gen).to(torch.bfloat16)
    w = (torch.randn(27, cout, cin, generator=gen) * 0.2).to(torch.bfloat16)
    bias = torch.randn(cout, generator=gen)
    w5 = w.double().reshape(3, 3, 3, cout, cin).permute(3, 4, 0, 1, 2).contiguous()
    x5 = x.double().permute(0, 4, 1, 2, 3).contiguous()
    conv = torch.nn.functional.conv3d
    ref = conv(x5, w5, bias.double(), padding=1).permute(0, 2, 3, 4, 1)
    mag = conv(x5.abs(), w5.abs(), bias.double().abs(), padding=1).permute(0, 2, 3, 4, 1)
    tol = 433 * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if cout == 16 else 0.0)
    xd, wd, bd = x.cuda(), w.cuda(), bias.cuda()
    dt = torch.bfloat16 if cout == 16 else torch.float32
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    n = ref.numel()
    for relu, shift in ((0, 0), (1, 0), (1, 1)):
        # shift: an output that is aligned to its element only; what lies around it stays
        buf = torch.full((n + 64,), 7.0, dtype=dt, device="cuda")
        out = buf[32 + shift:32 + shift + n]
        rc = _lib.lib().np_net_conv3d_fwd_mfma(p(xd), cin, p(wd), p(bd), cout, relu, B, Z, Y, X, p(out), None)
        torch.cuda.synchronize()
        assert rc == 0
        got = out.double().cpu().reshape(ref.shape)
        want = ref.clamp(min=0.0) if relu else ref
        assert ((got - want).abs() <= tol).all()
        assert (buf[:32 + shift] == 7.0).all() and (buf[32 + shift + n:] == 7.0).all()
