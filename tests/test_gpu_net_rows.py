"""Inference layers on rows longer than a buffer's 2^31 bytes (2^26 voxels and more), at both ends and
around voxel 2^26, against FP64 convolutions of the same bfloat16 inputs and weights.

Tolerance: 27 cin products and the bias in FP32, each addition within 2^-24 of the sum of the magnitudes S:
433 x 2^-24 S; a bfloat16 output adds 2^-8 of the value.
"""
import ctypes

import pytest
import torch

from paper_2001_02327_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout", [(2, 16), (16, 16), (16, 1)])
def test_long_row(cin, cout):
    X, period = (1 << 26) + 40, 1 << 16
    gen = torch.Generator().manual_seed(cin + cout)
    one = torch.randn(period, cin, generator=gen).to(torch.bfloat16)
    w = (torch.randn(27, cout, cin, generator=gen) * 0.2).to(torch.bfloat16)
    bias = torch.randn(cout, generator=gen)
    x = one.cuda().repeat((X + period - 1) // period, 1)[:X].contiguous()
    out = torch.empty((X, cout), dtype=torch.bfloat16 if cout == 16 else torch.float32, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    wd, bd = w.cuda(), bias.cuda()
    rc = _lib.lib().np_net_conv3d_fwd_mfma(p(x), cin, p(wd), p(bd), cout, 0, 1, 1, 1, X, p(out), None)
    torch.cuda.synchronize()
    assert rc == 0
    k = w.double()[12:15].permute(1, 2, 0).contiguous()  # the row's own taps (dz = dy = 0)
    for lo, hi in ((0, 3000), ((1 << 26) - 1500, X)):
        a, b = max(lo - 1, 0), min(hi + 1, X)
        v = x[a:b].cpu().double().t().unsqueeze(0).contiguous()
        conv = lambda u, q, c: torch.nn.functional.conv1d(u, q, c, padding=1)[0].t()[lo - a:hi - a]  # noqa: E731
        ref, mag = conv(v, k, bias.double()), conv(v.abs(), k.abs(), bias.double().abs())
        tol = 433 * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if cout == 16 else 0.0)
        assert ((out[lo:hi].cpu().double() - ref).abs() <= tol).all()
