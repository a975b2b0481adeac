"""Timing cases of the nested Poisson solver and of its guess network.

A case is a dict of plain values.  `listed()` names the cases that are always
measured, `draw(rng)` gives one more of the same ranges, `prepare` makes what a
program holds before the call (inputs, solver handle, output arrays, network
state) on the GPU, `run` makes one pass through the public entry points,
`work` counts the bytes and operations a pass cannot do without, and `exact`
gives the same outputs in plain FP64 torch: every nested level solved directly
by diagonalising its Dirichlet Laplacian, the network by FP64 convolutions.

Kinds of cases
  solve   one nested solve and the forces on every patch (optionally the
          potentials too), the step of a self-gravitating hydrodynamics code;
  train   one Adam step of the guess network on one level's sample, the step
          of training a new network;
  layers  the three network layers on the matrix cores, each on its own
          bfloat16 input: the inference a learned guess pays for per level.
"""
import ctypes
import math
import random

import numpy as np
import torch

from paper_2001_02327_amd import _lib, learned
from paper_2001_02327_amd import workloads as W
from paper_2001_02327_amd.solver import NestedPoissonSolver

# solver settings by the name a case gives them: the paper's FP64 V(2,1) (the
# default of the library), the two mixed-precision solves with adaptive inner
# cycles, and the benchmark's fastest schedule of each storage type
SETTINGS = {
    "fp64": dict(precision="fp64"),
    "fp64_v11": dict(precision="fp64", n_pre=1, n_post=1),
    "fp32": dict(precision="fp32_dc", inner_cycles="adaptive"),
    "fp32_v11": dict(precision="fp32_dc", inner_cycles="adaptive", n_pre=1, n_post=1),
    "fp16": dict(precision="fp16s_dc", inner_cycles="adaptive"),
    "fp16_v112": dict(precision="fp16s_dc", inner_cycles="adaptive", n_pre=1, n_post=1, coarse_post=2),
}


def _solve(name, workload, size, levels=0, settings="fp64", stop="residual", guess="interp", potentials=False, **more):
    c = dict(kind="solve", workload=workload, size=size, levels=levels, settings=settings, stop=stop, guess=guess,
             potentials=potentials, **more)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: a 2-D test problem, every launch tiny (latency)
        _solve("gauss2d_2x64_fp64", "gauss2d", 64, 2),
        # the paper's 2-D problem at its largest size, with the paper's stop rule
        _solve("paper2d_4x1024_delta", "paper2d", 1024, 4, stop="force_delta"),
        # an ordinary 3-D solve with the library's defaults
        _solve("plummer_3x128_fp64", "plummer", 128, 3),
        # a larger stack around an off-centre sphere, FP32 inner cycles
        _solve("offset_4x256_fp32", "plummer_offset", 256, 4, "fp32"),
        # the benchmark workload in its fastest setting and in plain FP64 (the largest)
        _solve("two_plummer_5x512_fp16", "two_plummer", 512, 5, "fp16_v112"),
        _solve("two_plummer_5x512_fp64", "two_plummer", 512, 5),
        # patch-based refinement: eight 64^3 patches solved as one batch under a 256^3 base
        _solve("many_256_8x64_fp64", "many", 256),
        # non-cubic patches of ragged sizes (256 x 128 x 184 base), potentials for an energy diagnostic
        _solve("box_256_fp16", "box", 4, settings="fp16", potentials=True),
        # one GPU's share of a 512^3 level split eight ways
        _solve("slab_512x512x64_fp16", "slab", 512, settings="fp16_v112"),
        # the learned initial guess run on every refined level of every solve
        _solve("learned_3x128_fp32", "plummer", 128, 3, "fp32", guess="learned"),
        # one training step at the size the shipped weights were trained at
        dict(name="train_130", kind="train", z=130, y=130, x=130),
        # inference of the three layers on a 256^3 patch with its inner buffer layer
        dict(name="layers_258", kind="layers", z=258, y=258, x=258),
    ]


def _log_even(rng, lo, hi, step):
    """A multiple of `step` between lo and hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, step * int(round(v / step))))


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _accepted(case):
    """Whether the library takes the case's geometry (some sizes give a hierarchy it refuses)."""
    try:
        _lib.plan(_lib.make_config(_geometry(case), **SETTINGS[case["settings"]]))
    except (_lib.NestedPoissonError, ValueError):
        return False
    return True


def draw(rng):
    kind = rng.choices(["solve2d", "solve3d", "many", "box", "slab", "learned", "train", "layers"],
                       [2, 3, 1, 2, 1, 1, 2, 1])[0]
    if kind == "train":
        return dict(kind="train", z=_log_int(rng, 18, 130), y=_log_int(rng, 18, 130), x=_log_int(rng, 18, 130))
    if kind == "layers":
        return dict(kind="layers", z=_log_int(rng, 18, 258), y=_log_int(rng, 18, 258), x=_log_int(rng, 18, 258))
    while True:
        mixed = rng.choice(["fp64", "fp64_v11", "fp32", "fp32_v11", "fp16", "fp16_v112"])
        if kind == "solve2d":
            if rng.random() < 0.5:
                c = _solve("", "gauss2d", _log_even(rng, 32, 1024, 4), 2, rng.choice(["fp64", "fp64_v11", "fp32"]))
            else:
                c = _solve("", "paper2d", _log_even(rng, 32, 1024, 4), rng.randint(2, 4),
                           rng.choice(["fp64", "fp32"]), stop="force_delta")
        elif kind == "solve3d":
            c = _solve("", rng.choice(["plummer", "plummer_offset", "two_plummer"]), _log_even(rng, 16, 320, 4),
                       rng.randint(2, 4), mixed, potentials=rng.random() < 0.3)
        elif kind == "many":
            c = _solve("", "many", _log_even(rng, 64, 256, 16))
        elif kind == "box":
            n = [_log_even(rng, 24, 256, 2) for _ in range(3)]
            m = [max(8, 2 * rng.randint(n[a] // 4, n[a] * 3 // 4)) for a in range(3)]
            m = [min(m[a], 2 * n[a] - 8) for a in range(3)]
            c = _solve("", "box2", 0, settings=mixed, potentials=rng.random() < 0.3, nx=n[0], ny=n[1], nz=n[2],
                       mx=m[0], my=m[1], mz=m[2])
        elif kind == "slab":
            c = _solve("", "slab", _log_even(rng, 128, 512, 16), settings=mixed)
        else:
            c = _solve("", "plummer", _log_even(rng, 32, 192, 4), rng.randint(2, 3), rng.choice(["fp32", "fp16"]),
                       guess="learned")
        if _accepted(c):
            return c


# ------------------------------------------------------------------ inputs
def _geometry(case):
    w, n, lev = case["workload"], case["size"], case["levels"]
    if w == "gauss2d":
        return W.c1_gaussian_2d(n).geom
    if w == "paper2d":
        return W.paper2d(n, lev).geom
    if w in ("plummer", "plummer_offset", "two_plummer"):
        return W.centred_geometry(3, lev, n, 1.0, 1.0)
    if w == "many":
        return W.many_patches_3d(n, 2).geom
    if w == "box":
        return W.box_plummer_3d(n).geom
    if w == "box2":
        e, m = (case["nx"], case["ny"], case["nz"]), (case["mx"], case["my"], case["mz"])
        return W.box_geometry(3, e, m, tuple((e[a] - m[a] // 2) // 2 for a in range(3)), dx0=2.0 / max(e))
    if w == "slab":
        return W.slab_two_plummer(n).geom
    raise ValueError(w)


def _problem(case, geom, seed):
    """The workload's density with its masses, radii, widths and centres moved a little by the seed."""
    r = random.Random(int(seed))
    jit = lambda v, by: v * r.uniform(1.0 - by, 1.0 + by)  # noqa: E731
    w = case["workload"]
    if w == "gauss2d":
        return W.Gaussian(jit(0.1, 0.1), 1.0)
    if w == "paper2d":
        return W.Paper2D(jit(0.3, 0.1))
    if w == "plummer":
        sph = [(1.0, 0.05, (0.0, 0.0, 0.0))]
    elif w == "plummer_offset":
        sph = [(1.0, 0.02, (0.1, -0.05, 0.03))]
    elif w in ("two_plummer", "slab"):
        sph = [(1.0, 0.03, (0.0, 0.0, 0.0)), (0.3, 0.015, (0.2, 0.0, 0.0))]
    else:
        leaves = [l for l in range(geom.nlevels) if not geom.children(l)]
        a = 0.04 if w == "many" else 0.06 * max(geom.ext(0)) * geom.dx0
        sph = [(1.0, a, tuple(geom.lo(l)[k] + 0.5 * geom.ext(l)[k] * geom.dx(l) for k in range(3))) for l in leaves]
    d = 0.2 * min(a for _, a, _ in sph)
    return W.Plummer([(jit(M, 0.2), jit(a, 0.1), tuple(v + r.uniform(-d, d) for v in c)) for M, a, c in sph])


def _inputs(case, seed):
    geom = _geometry(case)
    prob = _problem(case, geom, seed)
    return geom, W.make_inputs(geom, prob, device="cuda")


def _features(case, seed):
    """A training sample [1, Z, Y, X, 2] FP32 on Gamma of a refined patch: f / max|f| and the residual of the
    potential interpolated from the parent level / max|f|, for one to eight Plummer spheres whose radii are 5 to
    20 cells, as on the refined levels of the training workload."""
    shape = [case["z"], case["y"], case["x"]]
    n1 = [max(8, (v - 2) // 2 * 2) for v in reversed(shape)]          # the patch, even per axis
    n0 = [v // 2 + 2 * max(2, v // 8) + (v // 2) % 2 for v in n1]
    off = [(n0[a] - n1[a] // 2) // 2 for a in range(3)]
    g = W.box_geometry(3, n0, n1, off, dx0=1.0 / max(n0))
    r = random.Random(int(seed))
    mid = [0.5 * n0[a] * g.dx0 for a in range(3)]
    sph = [(math.exp(r.gauss(0.0, 0.5)), r.uniform(5.0, 20.0) * g.dx(1),
            tuple(mid[a] * (1.0 + r.uniform(-0.4, 0.4)) for a in range(3))) for _ in range(r.randint(1, 8))]
    rho, po = W.make_inputs(g, W.Plummer(sph), device="cuda")
    phi0, f0 = _direct_level0(g, rho[0], po)
    phi1, f1 = _fill(g, 1, phi0, f0, rho[1])
    h = g.dx(1)
    c = phi1[1:-1, 1:-1, 1:-1]
    lap = (phi1[1:-1, 1:-1, :-2] + phi1[1:-1, 1:-1, 2:] + phi1[1:-1, :-2, 1:-1] + phi1[1:-1, 2:, 1:-1] +
           phi1[:-2, 1:-1, 1:-1] + phi1[2:, 1:-1, 1:-1] - 6.0 * c) / (h * h)
    f = f1[1:-1, 1:-1, 1:-1]
    x = torch.stack([f, f - lap], dim=-1) / f.abs().max()
    out = torch.zeros(shape + [2], dtype=torch.float64, device="cuda")  # odd sizes: zeros past the patch
    k = [min(shape[a], x.shape[a]) for a in range(3)]
    out[:k[0], :k[1], :k[2]] = x[:k[0], :k[1], :k[2]]
    return out.to(torch.float32).unsqueeze(0).contiguous()


def _adam_state(seed):
    """First and second moments as they are some way into a training run."""
    r = np.random.default_rng(int(seed))
    n = learned.n_params()
    v = 1e-8 * np.exp(r.normal(0.0, 1.0, n))
    return (np.sqrt(v) * 0.1 * r.standard_normal(n)).astype(np.float32), v.astype(np.float32)


def _layer_inputs(case, seed):
    """bfloat16 inputs of the three layers: features, and two rectified hidden activations; weights and biases."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    s = (1, case["z"], case["y"], case["x"])
    x = [torch.randn(s + (ci,), generator=gen, device="cuda") * (0.1 if ci == 2 else 0.3)
         for ci, _ in learned.LAYERS]
    x = [t if k == 0 else t.clamp_min_(0.0) for k, t in enumerate(x)]
    return [t.to(torch.bfloat16) for t in x], _params(torch.from_numpy(learned.load_weights()).cuda())


def _params(theta):
    """[(bfloat16 weights [27][cout][cin], FP32 bias)] of a parameter vector."""
    out, k = [], 0
    for ci, co in learned.LAYERS:
        nw = 27 * ci * co
        out.append((theta[k:k + nw].to(torch.bfloat16).contiguous(), theta[k + nw:k + nw + co].contiguous()))
        k += nw + co
    return out


def prepare(case, seed):
    if case["kind"] == "train":
        net = learned.GuessNet(learned.load_weights())
        m, v = _adam_state(seed)
        net.m.copy_(torch.from_numpy(m))
        net.v.copy_(torch.from_numpy(v))
        net.step = 1000
        return dict(kind="train", net=net, x=_features(case, seed))
    if case["kind"] == "layers":
        xs, par = _layer_inputs(case, seed)
        outs = [torch.empty(x.shape[:4] + (co,), dtype=torch.bfloat16 if co == 16 else torch.float32, device="cuda")
                for x, (_, co) in zip(xs, learned.LAYERS)]
        return dict(kind="layers", xs=xs, par=par, outs=outs)
    geom, (rho, po) = _inputs(case, seed)
    kw = dict(SETTINGS[case["settings"]], stop_rule=case["stop"])
    if case["guess"] == "learned":
        kw.update(guess="learned", guess_gate=False)
    s = NestedPoissonSolver(geom, **kw)
    if case["guess"] == "learned":
        s.set_guess_weights(learned.load_weights())
    new = lambda l, pad: torch.empty(geom.shape(l, pad), dtype=torch.float64, device="cuda")  # noqa: E731
    return dict(kind="solve", solver=s, rho=rho, po=po, geom=geom,
                F=[[new(l, 0) for _ in range(geom.dim)] for l in range(geom.nlevels)],
                phi=[new(l, 2) for l in range(geom.nlevels)] if case["potentials"] else [])


def run(state):
    if state["kind"] == "train":
        net = state["net"]
        loss = net.train_step_residual(state["x"], lr=2e-4)
        return dict(loss=loss, grad=net.grad, theta=net.theta)
    if state["kind"] == "layers":
        L, st = _lib.lib(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        for k, (ci, co) in enumerate(learned.LAYERS):
            x, (w, b), out = state["xs"][k], state["par"][k], state["outs"][k]
            B, Z, Y, X, _ = x.shape
            rc = L.np_net_conv3d_fwd_mfma(ctypes.c_void_p(x.data_ptr()), ci, ctypes.c_void_p(w.data_ptr()),
                                          ctypes.c_void_p(b.data_ptr()), co, int(k < 2), B, Z, Y, X,
                                          ctypes.c_void_p(out.data_ptr()), st)
            if rc:
                raise _lib.NestedPoissonError(rc, "conv3d_fwd_mfma")
        return state["outs"]
    s = state["solver"]
    s.solve(state["rho"], state["po"])
    out = dict(F=[s.forces(l, out=state["F"][l]) for l in range(state["geom"].nlevels)])
    if state["phi"]:
        out["phi"] = [s.potential(l, out=state["phi"][l]) for l in range(state["geom"].nlevels)]
    return out


def work(case):
    if case["kind"] in ("train", "layers"):
        nv = float(case["z"] * case["y"] * case["x"])
        macs = sum(27.0 * ci * co for ci, co in learned.LAYERS) * nv
        if case["kind"] == "layers":
            return dict(bytes=nv * (2 * (2 + 16 + 16) + 2 * (16 + 16) + 4), flops=2.0 * macs)
        # forward, weight gradient and (below the first layer) data gradient
        first = 27.0 * 2 * 16 * nv
        return dict(bytes=nv * 8 + 5 * 4 * learned.n_params(), flops=2.0 * (3 * macs - first))
    g = _geometry(case)
    d, b, pts = g.dim, 0.0, 0.0
    for l in range(g.nlevels):
        cells = float(np.prod(g.shape(l)))
        pts += float(np.prod(g.shape(l, 1)))
        b += 8.0 * (float(np.prod(g.shape(l, 1 if l == 0 else 0))) + d * cells)
        if case["potentials"]:
            b += 8.0 * float(np.prod(g.shape(l, 2)))
    b += 8.0 * (float(np.prod(g.shape(0, 2))) - float(np.prod(g.shape(0, 1))))
    # about ten cycles to 1e-10, each three sweeps and a residual of 2d + 2 operations per point (8/7 of them)
    return dict(bytes=b, flops=10.0 * 4.0 * (2 * d + 2) * pts * 8.0 / 7.0)


# ------------------------------------------------------------------ the same outputs in plain FP64 torch
def _along(a, m, axis):
    """m applied to `a` along one axis."""
    t = a.movedim(axis, 0)
    s = t.shape
    r = m @ t.reshape(s[0], -1).contiguous()
    return r.reshape((m.shape[0],) + tuple(s[1:])).movedim(0, axis).contiguous()


def _sine(n):
    """Eigenvectors (orthonormal, symmetric) and eigenvalues of the 1-D Dirichlet second difference on n points."""
    k = torch.arange(1, n + 1, dtype=torch.float64, device="cuda")
    m = torch.sin(math.pi / (n + 1) * ((k[:, None] * k[None, :]) % (2 * (n + 1)))) * math.sqrt(2.0 / (n + 1))
    return m, -4.0 * torch.sin(math.pi * k / (2.0 * (n + 1))) ** 2


def _inner(d, lo=1):
    return tuple(slice(lo, -lo) for _ in range(d))


def _dirichlet(phi, f, h):
    """phi with its interior replaced by the solution of the (2d+1)-point equation lap phi = f (f: interior)."""
    d = phi.dim()
    b = f * (h * h)
    for ax in range(d):
        lo = [slice(1, -1)] * d
        hi = [slice(1, -1)] * d
        lo[ax], hi[ax] = 0, -1
        b.select(ax, 0).sub_(phi[tuple(lo)])
        b.select(ax, b.shape[ax] - 1).sub_(phi[tuple(hi)])
    lam = 0.0
    mats = []
    for ax in range(d):
        m, e = _sine(b.shape[ax])
        mats.append(m)
        lam = lam + e.reshape([-1 if a == ax else 1 for a in range(d)])
        b = _along(b, m, ax)
    b = b / lam
    for ax in range(d):
        b = _along(b, mats[ax], ax)
    out = phi.clone()
    out[_inner(d)] = b
    return out


def _direct_level0(g, rho0, po):
    f = torch.zeros(g.shape(0, 2), dtype=torch.float64, device="cuda")
    f[_inner(g.dim)] = 4.0 * math.pi * g.G * rho0
    return _dirichlet(po.clone(), f[_inner(g.dim)].clone(), g.dx(0)), f


def _fill(g, l, phip, fp, rho):
    """Padded potential interpolated from the parent and right-hand side of level l (inner layer interpolated)."""
    d, p = g.dim, g.par(l)
    phi, fi = phip, fp
    for ax in range(d):  # tensor axis ax is x for the last one
        a = d - 1 - ax
        n = g.ext(l)[a]
        m = torch.zeros(n + 4, g.ext(p)[a] + 4, dtype=torch.float64)
        for q in range(n + 4):
            i = q - 2
            par = g.off[l][a] + i // 2
            nb = par - 1 if i % 2 == 0 else par + 1
            m[q, par + 2] = 0.75
            m[q, nb + 2] = 0.25
        m = m.cuda()
        phi, fi = _along(phi, m, ax), _along(fi, m, ax)
    f = torch.zeros_like(fi)
    f[_inner(d)] = fi[_inner(d)]
    f[_inner(d, 2)] = 4.0 * math.pi * g.G * rho
    return phi, f


def _forces(phi, dx):
    d = phi.dim()
    out = []
    for a in range(d):
        ax = d - 1 - a

        def sh(k):
            s = [slice(2, -2)] * d
            s[ax] = slice(2 + k, phi.shape[ax] - 2 + k)
            return phi[tuple(s)]
        out.append(-(8.0 * (sh(1) - sh(-1)) - (sh(2) - sh(-2))) / (12.0 * dx))
    return out


def _conv64(x, w, b, co):
    """x [1, Z, Y, X, cin] FP64, w [27][cout][cin]: same-size zero-padded convolution, taps added one by one."""
    _, Z, Y, X, ci = x.shape
    w = w.double().reshape(27, co, ci)
    pad = torch.zeros(Z + 2, Y + 2, X + 2, ci, dtype=torch.float64, device=x.device)
    pad[1:-1, 1:-1, 1:-1] = x[0]
    out = b.double().expand(Z * Y * X, co).clone()
    for t in range(27):
        dz, dy, dx = t // 9, t // 3 % 3, t % 3
        out += pad[dz:dz + Z, dy:dy + Y, dx:dx + X].reshape(-1, ci) @ w[t].t().contiguous()
    return out.reshape(1, Z, Y, X, co)


def _lap64(a):
    p = torch.nn.functional.pad(a, (1, 1, 1, 1, 1, 1))
    c = p[1:-1, 1:-1, 1:-1]
    return (p[1:-1, 1:-1, :-2] + p[1:-1, 1:-1, 2:] + p[1:-1, :-2, 1:-1] + p[1:-1, 2:, 1:-1] + p[:-2, 1:-1, 1:-1] +
            p[2:, 1:-1, 1:-1] - 6.0 * c)


def _exact_train(case, seed):
    bf = lambda t: t.to(torch.float32).to(torch.bfloat16).double()  # noqa: E731
    theta = torch.from_numpy(learned.load_weights()).cuda()
    par = _params(theta)
    acts = [bf(_features(case, seed))]
    for k, (ci, co) in enumerate(learned.LAYERS):
        y = _conv64(acts[-1], par[k][0], par[k][1], co)
        acts.append(bf(y.clamp_min(0.0)) if k < 2 else y)
    r = acts[0][0, ..., 1]
    d = _lap64(acts[3][0, ..., 0]) - r
    n = float(d.numel())
    loss = (d * d).sum() / n
    g = _lap64(2.0 * d / n)[None, ..., None]
    grads = [None] * 3
    Z, Y, X = case["z"], case["y"], case["x"]
    for k in (2, 1, 0):
        ci, co = learned.LAYERS[k]
        a = torch.zeros(Z + 2, Y + 2, X + 2, ci, dtype=torch.float64, device="cuda")
        a[1:-1, 1:-1, 1:-1] = acts[k][0]
        gp = torch.zeros(Z + 2, Y + 2, X + 2, co, dtype=torch.float64, device="cuda")
        gp[1:-1, 1:-1, 1:-1] = g[0]
        gt = g.reshape(-1, co).t().contiguous()
        gw, w = [], par[k][0].double().reshape(27, co, ci)
        gin = torch.zeros(Z * Y * X, ci, dtype=torch.float64, device="cuda")
        for t in range(27):
            dz, dy, dx = t // 9, t // 3 % 3, t % 3
            gw.append(gt @ a[dz:dz + Z, dy:dy + Y, dx:dx + X].reshape(-1, ci))
            gin += gp[2 - dz:2 - dz + Z, 2 - dy:2 - dy + Y, 2 - dx:2 - dx + X].reshape(-1, co) @ w[t]
        grads[k] = torch.cat([torch.stack(gw).reshape(-1), gt.sum(1)])
        g = (gin.reshape(1, Z, Y, X, ci) * (acts[k] > 0)) if k else None
    g = torch.cat(grads)
    m, v = (torch.from_numpy(t).cuda().double() for t in _adam_state(seed))
    f32 = lambda t: float(np.float32(t))  # noqa: E731
    b1, b2, step = f32(0.9), f32(0.999), 1001
    m = b1 * m + (1.0 - b1) * g
    v = b2 * v + (1.0 - b2) * g * g
    th = theta.double() - f32(2e-4) * (m / (1.0 - b1 ** step)) / ((v / (1.0 - b2 ** step)).sqrt() + f32(1e-8))
    return dict(loss=loss.reshape(1), grad=g, theta=th)


def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] == "layers":
        xs, par = _layer_inputs(case, seed)
        out = []
        for k, (ci, co) in enumerate(learned.LAYERS):
            y = _conv64(xs[k].double(), par[k][0], par[k][1], co)
            out.append(y.clamp_min(0.0) if k < 2 else y)
        return out
    g, (rho, po) = _inputs(case, seed)
    phi, f, F = [], [], []
    for l in range(g.nlevels):
        if l == 0:
            p, fl = _direct_level0(g, rho[0], po)
        else:
            p, fl = _fill(g, l, phi[g.par(l)], f[g.par(l)], rho[l])
            p = _dirichlet(p, fl[_inner(g.dim)].clone(), g.dx(l))
        phi.append(p)
        f.append(fl)
        F.append(_forces(p, g.dx(l)))
    return dict(F=F, phi=phi) if case["potentials"] else dict(F=F)
