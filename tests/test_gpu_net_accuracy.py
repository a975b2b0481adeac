"""Weight and bias gradients of the training layers on a large volume: no further from 64 bits than the sums over
voxel rows (k_conv_bwd_weight_part), which calls with arrays off a 16-byte boundary take.

Both are FP32 sums of 2 N products of 258^3 voxels; the rows are summed in two stages of 64 and a thousand, so a
single running sum over a workgroup's range (2256 products deep there) loses to them on gradients of either sign.
"""
import ctypes

import pytest
import torch

from paper_2001_02327_amd import _lib, learned

pytestmark = pytest.mark.gpu


def _p(t):
    return ctypes.c_void_p(t.data_ptr())


def _reference(x, g):
    n, ci, co = x.shape[1], x.shape[-1], g.shape[-1]
    xp = torch.zeros((n + 2,) * 3 + (ci,), dtype=torch.float64, device="cuda")
    xp[1:-1, 1:-1, 1:-1] = x[0].double()
    gt = g[0].double().reshape(n, n * n, co).transpose(1, 2).contiguous()  # plane by plane
    taps = [(t // 9, t // 3 % 3, t % 3) for t in range(27)]
    w = torch.stack([torch.bmm(gt, xp[a:a + n, b:b + n, c:c + n].reshape(n, n * n, ci).contiguous()).sum(0)
                     for a, b, c in taps])
    return w.reshape(-1), gt.sum((0, 2))


def _gradients(x, g, off):
    n, ci, co = x.shape[1], x.shape[-1], g.shape[-1]
    L = _lib.lib()
    if off:
        x, g = (torch.cat([t.new_zeros(1), t.reshape(-1)])[1:] for t in (x, g))
    ws = L.np_net_workspace_bytes(ci, co, 0)
    work = torch.empty(ws // 4 + 1, device="cuda")
    gw, gb = torch.empty(27 * co * ci, device="cuda"), torch.empty(co, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.np_net_conv3d_bwd_weight(_p(x), ci, _p(g), co, 1, n, n, n, _p(gw), _p(gb), _p(work), ws, st) == 0
    torch.cuda.synchronize()
    return gw.double(), gb.double()


@pytest.mark.parametrize("ci,co", learned.LAYERS)
def test_large_volume(ci, co):
    n = 258
    gen = torch.Generator(device="cuda").manual_seed(n + ci)
    x = torch.randn((1, n, n, n, ci), generator=gen, device="cuda")
    g = torch.randn((1, n, n, n, co), generator=gen, device="cuda")
    if ci == 16:
        x.clamp_(min=0.0)
    ref = _reference(x, g)
    blocks, rows = _gradients(x, g, False), _gradients(x, g, True)
    for k in range(2):
        err = [float((v[k] - ref[k]).abs().max() / ref[k].abs().max()) for v in (blocks, rows)]
        print("%d -> %d %s: blocks %.2e, rows %.2e" % (ci, co, ("weights", "bias")[k], *err), flush=True)
        assert err[0] <= err[1]
