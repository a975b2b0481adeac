"""The training convolutions on the FP32 matrix cores (the network's layer
shapes, 16-byte aligned arrays) against the thread-per-voxel kernels, which
take every other call: arrays four bytes off a 16-byte boundary go to those.

Forward: the same chain of FP32 fused multiply-adds, so the same bits.
Gradients: FP32 sums in another order, at most 27 * 16 = 432 terms per value
(data) or one per voxel (weights): 1e-5 of the largest value.  A value that is
not finite in an input, a weight or an output gradient reaches the same
outputs as the same kind of value.
"""
import ctypes

import pytest
import torch

from paper_2001_02327_amd import _lib, learned

pytestmark = pytest.mark.gpu

# one voxel, one whole block, a voxel past a block on each axis, ragged rows, few-channel blocks of 32 x 8 x 8 and one past them
SHAPES = [(1, 1, 1, 1), (1, 4, 4, 16), (2, 5, 3, 17), (1, 2, 9, 33), (1, 9, 8, 32), (1, 10, 5, 50), (3, 6, 7, 15)]


@pytest.fixture(autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need the MI355X"


def _p(t):
    return ctypes.c_void_p(t.data_ptr() if t is not None else 0)


def _off(t):
    """A copy of t four bytes past a 16-byte boundary."""
    b = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    b[1:].copy_(t.reshape(-1))
    return b[1:].view(t.shape)


def _off_w(w):
    """A copy of the weights two bytes past a 4-byte boundary (the few-channel kernel takes aligned ones)."""
    b = torch.empty(w.numel() + 1, dtype=w.dtype, device=w.device)
    b[1:].copy_(w)
    return b[1:]


def _run(x, w, b, g, act, general):
    """(forward, rounded forward, data gradient, masked data gradient, weight gradient, bias gradient)."""
    L, st = _lib.lib(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    B, Z, Y, X, ci = x.shape
    co = g.shape[-1]
    if general:
        x, g, w, act = _off(x), _off(g), _off_w(w), _off(act)
    new = (lambda s: _off(torch.zeros(s, device="cuda"))) if general else (lambda s: torch.zeros(s, device="cuda"))
    y, yr, gi, gm = new(g.shape), new(g.shape), new(x.shape), new(x.shape)
    gw, gb = torch.zeros(27 * co * ci, device="cuda"), torch.zeros(co, device="cuda")
    ws = L.np_net_workspace_bytes(ci, co, 0)
    work = torch.empty(ws // 4 + 1, device="cuda")
    assert L.np_net_conv3d_fwd(_p(x), ci, _p(w), _p(b), co, 0, B, Z, Y, X, _p(y), st) == 0
    assert L.np_net_conv3d_fwd_round(_p(x), ci, _p(w), _p(b), co, B, Z, Y, X, _p(yr), st) == 0
    assert L.np_net_conv3d_bwd_data(_p(g), co, _p(w), ci, B, Z, Y, X, _p(gi), st) == 0
    assert L.np_net_conv3d_bwd_data_relu(_p(g), co, _p(w), ci, B, Z, Y, X, _p(act), _p(gm), st) == 0
    assert L.np_net_conv3d_bwd_weight(_p(x), ci, _p(g), co, B, Z, Y, X, _p(gw), _p(gb), _p(work), ws, st) == 0
    return [t.reshape(-1).clone() for t in (y, yr, gi, gm, gw, gb)]


def _inputs(shape, ci, co, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    w = (rnd((27 * co * ci,)) * 0.2).to(torch.bfloat16)
    return rnd(shape + (ci,)), w, rnd((co,)), rnd(shape + (co,)), rnd(shape + (ci,))


def _check(new, old):
    for k, (a, b) in enumerate(zip(new, old)):
        assert torch.equal(torch.isnan(a), torch.isnan(b)), k
        fin = torch.isfinite(b)
        assert torch.equal(torch.isfinite(a), fin), k
        assert torch.equal(a[~fin & ~torch.isnan(b)], b[~fin & ~torch.isnan(b)]), k
        if k < 2:
            assert torch.equal(a[fin], b[fin]), k
        elif fin.any():
            assert float((a[fin] - b[fin]).abs().max()) <= 1e-5 * float(b[fin].abs().max()), k


@pytest.mark.parametrize("ci,co", learned.LAYERS)
@pytest.mark.parametrize("shape", SHAPES)
def test_training_layers_match_the_general_kernels(shape, ci, co):
    x, w, b, g, act = _inputs(shape, ci, co, 7 * ci + co + sum(shape))
    _check(_run(x, w, b, g, act, False), _run(x, w, b, g, act, True))


@pytest.mark.parametrize("ci,co", learned.LAYERS)
@pytest.mark.parametrize("where", ["corner", "inside"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("what", ["input", "weight", "gradient"])
def test_training_layers_non_finite(what, value, where, ci, co):
    shape = (1, 6, 7, 19)
    x, w, b, g, act = _inputs(shape, ci, co, 11 * ci + co)
    at = (0, 0, 0, 18, 0) if where == "corner" else (0, 3, 4, 9, 0)
    if what == "input":
        x[at] = value
    elif what == "gradient":
        g[at] = value
    else:
        w[5 * co * ci if where == "corner" else 13 * co * ci] = value
    _check(_run(x, w, b, g, act, False), _run(x, w, b, g, act, True))
