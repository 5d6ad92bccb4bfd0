"""Performance cases of the library: what its users run, through the public Python entry points.

listed() names the cases, draw(rng) gives more of the same ranges, prepare(case, seed) makes what a
program holds before the call (fields, context, bound workspace, network with weights), run(state)
is one pass, work(case) the bytes and operations one pass cannot do without, exact(case, seed) the
same results from plain FP64 torch.

Kinds:
  step        one implicit Euler step, tbs_timestep (right-hand side, CG, FP64 check)
  apply       y = A u of one operator evaluation
  varcoef     y = F(u) with variable diffusion and absorption
  transform   samples -> coefficients (direct) and coefficients -> samples (indirect)
  net_forward the network's guess for one field
  net_train   one training step of the network (loss and gradient)
"""
import json
import math
import os

import numpy as np
import torch

import paper_1904_03057_amd as tbs

DEV = "cuda"
DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
ESZ = {"f64": 8, "f32": 4, "bf16": 2}
WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(tbs.__file__)), "weights", "guess_net_128")
RTOL = 1e-10      # the time step's default relative residual
GAMMA = 1e-3      # Robin / penalty parameter
PARAMS = [(2, 16), (16, 16), (16, 16), (16, 1)]


def _case(name, kind, grid, **kw):
    c = {"name": name} if name else {}
    c.update(kind=kind, nx=grid[0], ny=grid[1], nz=grid[2], **kw)
    return c


def listed():
    return [
        # the smallest step, where launches and host round trips are what counts: the 32^3 periodic
        # workload of the tests and of the graph-captured solves
        _case("step_f64_32", "step", (32, 32, 32), bc="periodic", degree=3, prec="fp64", lam=1.024, source=False),
        # a small box of ragged sizes with a source, refined FP32, even degree
        _case("step_mixed_ragged", "step", (131, 94, 61), bc="dirichlet", degree=2, prec="mixed", lam=3.0, source=True),
        # the ordinary step: the 256^3 workload with a Gaussian source, refined FP32
        _case("step_mixed_256", "step", (256, 256, 256), bc="dirichlet", degree=3, prec="mixed", lam=6.6, source=True),
        # the headline step: 928^3 (0.8e9 unknowns), refined FP32
        _case("step_mixed_928", "step", (928, 928, 928), bc="dirichlet", degree=3, prec="mixed", lam=8.63, source=False),
        # plain FP64 CG on the periodic grid of the degree sweep, highest degree
        _case("step_f64_n5", "step", (512, 256, 256), bc="periodic", degree=5, prec="fp64", lam=13.1, source=False),
        # a Robin / penalty box: its nearly empty corner functions make it ill-conditioned (hundreds of
        # iterations), so it is solved in FP64
        _case("step_robin", "step", (121, 104, 90), bc="robin", degree=3, prec="fp64", lam=4.0, source=True),
        # operator evaluations: the headline grid in FP32, and a ragged periodic one in FP64
        _case("apply_f32_928", "apply", (928, 928, 928), bc="dirichlet", degree=3, din="f32", dout="f32", lam=8.63),
        _case("apply_f64_ragged", "apply", (385, 259, 201), bc="periodic", degree=4, din="f64", dout="f64", lam=5.0),
        # variable coefficients (a heterogeneous medium), cubic
        _case("varcoef_f32", "varcoef", (192, 192, 192), bc="dirichlet", degree=3, din="f32", lam=6.6),
        # samples to coefficients and back
        _case("transform_256", "transform", (256, 256, 256), bc="dirichlet", degree=3),
        # the network's guess on a field of the evaluation range, and its training at its own grid and batch
        _case("net_forward_256", "net_forward", (256, 256, 256), bc="dirichlet", din="f64"),
        _case("net_train_128", "net_train", (128, 128, 128), bc="dirichlet", batch=4),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi, cap):
    while True:
        g = [_size(rng, lo, hi) for _ in range(3)]
        if rng.random() < 0.4:
            g[0] = max(lo, g[0] // 4 * 4)
        if g[0] * g[1] * g[2] <= cap:
            return g


def draw(rng):
    kind = rng.choice(["step", "step", "step", "apply", "apply", "varcoef", "transform", "net_forward", "net_train"])
    lam = round(rng.uniform(1.0, 13.0), 3)
    bc = rng.choice(["periodic", "dirichlet"])
    if kind == "step":
        source = rng.random() < 0.5
        if rng.random() < 0.15:
            return _case(None, kind, _grid(rng, 32, 200, 1 << 21), bc="robin", degree=rng.choice([1, 2, 3]), prec="fp64",
                         lam=lam, source=source)
        return _case(None, kind, _grid(rng, 32, 512, 1 << 25), bc=bc, degree=rng.choice([1, 2, 3, 3, 3, 4, 5]),
                     prec=rng.choice(["fp64", "mixed", "mixed"]), lam=lam, source=source)
    if kind == "apply":
        if rng.random() < 0.2:
            bc = "robin"
        din, dout = rng.choice([("f64", "f64"), ("f32", "f32"), ("bf16", "f32")])
        return _case(None, kind, _grid(rng, 32, 928, 1 << 28), bc=bc, degree=rng.choice([1, 2, 3, 3, 4, 5]), din=din,
                     dout=dout, lam=lam)
    if kind == "varcoef":
        return _case(None, kind, _grid(rng, 32, 256, 1 << 22), bc=bc, degree=rng.choice([1, 2, 3, 3, 4]),
                     din=rng.choice(["f32", "f32", "f64"]), lam=lam)
    if kind == "transform":
        return _case(None, kind, _grid(rng, 32, 512, 1 << 25), bc=bc, degree=rng.choice([2, 3, 3, 4, 5]))
    if kind == "net_forward":
        return _case(None, kind, _grid(rng, 32, 320, 1 << 24), bc=bc, din=rng.choice(["f64", "f32"]))
    return _case(None, kind, _grid(rng, 48, 160, 1 << 21), bc=bc, batch=rng.choice([1, 2, 4]))


# ------------------------------------------------------------------------------------------
# inputs


def _dims(c):
    return (c["nx"], c["ny"], c["nz"])


def _spacing(c):
    """One spacing for the three axes, the longest spanning the unit interval; tau = lam h^2."""
    h = 1.0 / (max(_dims(c)) + 1)
    return h, c.get("lam", 6.0) * h * h


def _gaussians(c, r, count, s_lo, s_hi, amp):
    """Sum of `count` Gaussians, centres in the middle 80 % of the box, FP64 on the GPU."""
    h, _ = _spacing(c)
    out = torch.zeros(c["nz"], c["ny"], c["nx"], dtype=torch.float64, device=DEV)
    x = [(np.arange(n) + 1.0) * h for n in _dims(c)]
    for _ in range(count):
        a, s = amp * r.standard_normal(), r.uniform(s_lo, s_hi)
        g = [np.exp(-(x[d] - r.uniform(0.1, 0.9) * x[d][-1]) ** 2 / (2 * s * s)) for d in range(3)]
        gx, gy, gz = (torch.from_numpy(v).to(DEV) for v in g)
        out.addcmul_((a * gz)[:, None, None] * gy[:, None], gx.expand(c["nz"], c["ny"], c["nx"]))
    return out


def _noise(c, r):
    """Periodic field: smoothed N(0,1) noise and four sine modes."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(r.integers(1 << 31)))
    u = torch.randn(c["nz"], c["ny"], c["nx"], dtype=torch.float64, device=DEV, generator=gen)
    for _ in range(2):
        for d in range(3):
            u = 0.5 * u + 0.25 * (u.roll(1, d) + u.roll(-1, d))
    z, y, x = (torch.arange(n, dtype=torch.float64, device=DEV) / n for n in u.shape)
    for _ in range(4):
        kx, ky, kz = (int(v) for v in r.integers(1, 5, 3))
        u += torch.sin(2 * math.pi * (kz * z[:, None, None] + ky * y[:, None] + kx * x))
    return u


def _field(c, r):
    return _noise(c, r) if c["bc"] == "periodic" else _gaussians(c, r, 16, 0.02, 0.1, 1.0)


def _source(c, r):
    return _gaussians(c, r, int(r.integers(1, 5)), 0.05, 0.15, 10.0)


def _coefficients(c, r):
    """Positive diffusion (of size tau) and absorption (of size 1) fields: smooth, with steep interfaces."""
    _, tau = _spacing(c)
    d = tau * (1.0 + 0.5 * torch.tanh(2.0 * _gaussians(c, r, 8, 0.05, 0.2, 2.0)))
    m = 1.0 + 0.5 * torch.tanh(_gaussians(c, r, 8, 0.05, 0.2, 1.0))
    return d, m


def _inputs(c, seed):
    """The case's inputs as FP64 fields already rounded to the type the call takes."""
    r = np.random.default_rng(seed)
    kind = c["kind"]
    if kind == "step":
        return [_field(c, r), _source(c, r) if c["source"] else None]
    if kind == "apply":
        return [_field(c, r).to(DTYPES[c["din"]])]
    if kind == "varcoef":
        u = _field(c, r)
        return [t.to(DTYPES[c["din"]]) for t in (u, *_coefficients(c, r))]
    if kind == "transform":
        return [_field(c, r)]
    if kind == "net_forward":
        return [t.to(DTYPES[c["din"]]) for t in (_field(c, r), _source(c, r))]
    # training pairs: fields, sources and an increment of the size a step gives, batch samples back to back
    _, tau = _spacing(c)
    u, q, du = [], [], []
    for _ in range(c["batch"]):
        a, f = _field(c, r), _source(c, r)
        u.append(a.float())
        q.append(f.float())
        du.append((tau * (_laplacian(a, c) + f)).float())
    return [torch.stack(v).contiguous() for v in (u, q, du)]


def _laplacian(a, c):
    """Second differences (zero or periodic continuation)."""
    h, _ = _spacing(c)
    per = c["bc"] == "periodic"
    lap = torch.zeros_like(a)
    for d in range(3):
        lap += _shift(a, d, 1, per) + _shift(a, d, -1, per) - 2 * a
    return lap / (h * h)


def _shift(a, d, k, per):
    """b[i] = a[i + k] along axis d, wrapped or continued by zeros."""
    if per:
        return a.roll(-k, d)
    out = torch.zeros_like(a)
    n = a.shape[d]
    if abs(k) < n:
        out.narrow(d, max(0, -k), n - abs(k)).copy_(a.narrow(d, max(0, k), n - abs(k)))
    return out


def _weights():
    """The repository's trained 128^3 network and its output scale."""
    with open(WEIGHTS + ".json") as f:
        meta = json.load(f)
    return np.fromfile(WEIGHTS + ".f32", dtype="<f4"), float(meta["out_scale"])


def _context(c):
    h, tau = _spacing(c)
    if c["kind"] == "transform":
        return tbs.Transform(_dims(c), c["degree"], c["bc"])
    if c["bc"] == "robin":
        return tbs.RobinContext(_dims(c), c["degree"], (h, h, h), tau, GAMMA)
    return tbs.Context(_dims(c), c["degree"], (h, h, h), tau, c["bc"])


PREC = {"fp64": tbs.PREC_FP64, "mixed": tbs.PREC_MIXED}


def prepare(case, seed):
    c = dict(case)
    s = {"c": c, "in": _inputs(c, seed)}
    shape = (c["nz"], c["ny"], c["nx"])
    if c["kind"] in ("net_forward", "net_train"):
        w, scale = _weights()
        train = c["kind"] == "net_train"
        net = tbs.Net()
        net.ensure_workspace(_dims(c), c.get("batch", 1), train)
        net.set_weights(w)
        # a late step of a decayed schedule: the trained network and a small learning rate
        net.set_hparams(out_scale=scale, lr=1e-6)
        s["net"] = net
        s["tau"] = _spacing(c)[1]
        if not train:
            s["out"] = torch.empty(shape, dtype=torch.float32, device=DEV)
        return s
    s["ctx"] = _context(c)
    if c["kind"] == "step":
        s["ctx"].ensure_workspace(PREC[c["prec"]])
        s["out"] = torch.empty(shape, dtype=torch.float64, device=DEV)
    elif c["kind"] == "transform":
        s["ctx"].ensure_workspace(tbs.PREC_FP64)
        s["coef"], s["out"] = torch.empty_like(s["in"][0]), torch.empty_like(s["in"][0])
    else:
        s["out"] = torch.empty(shape, dtype=DTYPES[c.get("dout", c["din"])], device=DEV)
    return s


def run(s):
    c, x = s["c"], s["in"]
    kind = c["kind"]
    if kind == "step":
        s["ctx"].timestep(x[0], x[1], s["out"], PREC[c["prec"]], RTOL, 5000)
        return s["out"]
    if kind == "apply":
        s["ctx"].apply(x[0], s["out"])
        return s["out"]
    if kind == "varcoef":
        s["ctx"].apply_varcoef(x[0], x[1], x[2], s["out"])
        return s["out"]
    if kind == "transform":
        s["coef"].copy_(x[0])
        s["ctx"].interp(x[0], s["coef"], 1e-12, 1000)
        s["ctx"].eval(s["coef"], s["out"])
        return {"coef": s["coef"], "samples": s["out"]}
    per = c["bc"] == "periodic"
    if kind == "net_forward":
        s["net"].forward(x[0], x[1], s["out"], per, s["tau"])
        return s["out"]
    loss = s["net"].train_step(x[0], x[1], x[2], c["batch"], per, s["tau"])
    return {"loss": loss, "grad": s["net"].get_grad()}


# ------------------------------------------------------------------------------------------
# what one pass cannot do without


def work(case):
    c = case
    N = c["nx"] * c["ny"] * c["nz"]
    kind = c["kind"]
    if kind == "step":
        # fields in and out once; the operations of one right-hand side, one operator and one check
        return {"bytes": 8.0 * N * (3 if c["source"] else 2), "flops": N * 3.0 * 7 * 2 * (2 * c["degree"] + 1)}
    if kind == "apply":
        return {"bytes": float(N * (ESZ[c["din"]] + ESZ[c["dout"]])), "flops": N * 7.0 * (3 * c["degree"] + 1)}
    if kind == "varcoef":
        # sum factorisation: interpolation of three fields (and the gradient) and the projection, per cell
        n, q = c["degree"], (3 * c["degree"] + 2) // 2
        fma = (n + 1) * (4 * q + 5 * q * q + 6 * q ** 3) + (n + 1) * (4 * q ** 3 + 3 * q * q + 2 * q) + 6 * q ** 3
        return {"bytes": 4.0 * N * ESZ[c["din"]], "flops": 2.0 * N * fma}
    if kind == "transform":
        # samples in, coefficients out; coefficients in, samples out
        return {"bytes": 4 * 8.0 * N, "flops": N * 2 * 3.0 * 2 * (2 * (c["degree"] // 2) + 1)}
    mac = 27.0 * sum(i * o for i, o in PARAMS)
    if kind == "net_forward":
        return {"bytes": N * (2.0 * ESZ[c["din"]] + 4), "flops": 2 * mac * N}
    b = c["batch"]
    return {"bytes": 12.0 * N * b, "flops": 2 * b * N * (3 * mac - 27.0 * 32)}


# ------------------------------------------------------------------------------------------
# the same in plain FP64: dense 1-D matrices of every axis, Kronecker products along the axes


def _bspline(p, x):
    x = -np.abs(np.asarray(x, dtype=np.float64))
    half = 0.5 * (p + 1)
    acc = np.zeros_like(x)
    for j in range(p + 2):
        t = x + half - j
        acc += (-1) ** j * math.comb(p + 1, j) * (np.where(t > 0, t, 0.0) ** p if p else (t > 0))
    return np.where(-x < half, acc / math.factorial(p), 0.0)


def _dbspline(p, x):
    x = np.asarray(x, dtype=np.float64)
    return _bspline(p - 1, x + 0.5) - _bspline(p - 1, x - 0.5)


def _band(taps, n, bc):
    """Symmetric banded matrix of one-sided taps: circulant (periodic) or truncated."""
    A = np.zeros((n, n))
    i = np.arange(n)
    for k in range(-(len(taps) - 1), len(taps)):
        if bc == "periodic":
            np.add.at(A, (i, (i + k) % n), taps[abs(k)])
        else:
            ok = (i + k >= 0) & (i + k < n)
            A[i[ok], i[ok] + k] += taps[abs(k)]
    return A


def _axis(c, n):
    """(M, W) of one axis: mass, and tau times stiffness (with the end terms of a Robin box)."""
    p = c["degree"]
    h, tau = _spacing(c)
    if c["bc"] != "robin":
        m = [_bspline(2 * p + 1, float(k)) for k in range(p + 1)]
        s = [-(_bspline(2 * p - 1, k + 1.0) - 2 * _bspline(2 * p - 1, float(k)) + _bspline(2 * p - 1, k - 1.0))
             for k in range(p + 1)]
        return _band(m, n, c["bc"]), tau / h ** 2 * _band(s, n, c["bc"])
    k = np.arange(n) - p // 2
    nc = n - 1 - 2 * (p // 2)
    g, w = np.polynomial.legendre.leggauss(p + 1)
    x = (np.arange(2 * nc)[:, None] * 0.5 + 0.25 + 0.25 * g).ravel()
    w = np.tile(0.25 * w, 2 * nc)
    B, D = _bspline(p, x[None] - k[:, None]), _dbspline(p, x[None] - k[:, None])
    e0, e1 = _bspline(p, -k.astype(float)), _bspline(p, (nc - k).astype(float))
    E = np.outer(e0, e0) + np.outer(e1, e1)
    return (B * w) @ B.T, tau * ((D * w) @ D.T / h ** 2 + E / (2 * GAMMA * h))


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _along(A, u, d):
    """A applied along x (d = 0), y (1) or z (2) of u[z][y][x]; A may be rectangular."""
    nz, ny, nx = u.shape
    if d == 0:
        return (u.reshape(-1, nx) @ A.T).reshape(nz, ny, -1)
    if d == 2:
        return (A @ u.reshape(nz, -1)).reshape(-1, ny, nx)
    out = torch.empty(nz, A.shape[0], nx, dtype=u.dtype, device=u.device)
    for z in range(nz):
        torch.mm(A, u[z], out=out[z])
    return out


def _exact_apply(c, u):
    M, W = zip(*((_gpu(m), _gpu(w)) for m, w in (_axis(c, n) for n in _dims(c))))
    ux = _along(M[0], u, 0)
    t = _along(M[1], _along(W[0], u, 0), 1)
    t += _along(W[1], ux, 1)
    ux = _along(M[1], ux, 1)
    y = _along(M[2], ux + t, 2)
    del t
    return y.add_(_along(W[2], ux, 2))


def _exact_step(c, u, q):
    """A^-1 M (u + tau q) in the eigenbasis of the axis pairs (W, M)."""
    _, tau = _spacing(c)
    g = u + tau * q if q is not None else u.clone()
    V, lam = [], []
    for n in _dims(c):
        m, w = _axis(c, n)
        L = np.linalg.cholesky(m)
        S = np.linalg.solve(L, np.linalg.solve(L, w).T)
        lv, Q = np.linalg.eigh(0.5 * (S + S.T))
        V.append(_gpu(np.linalg.solve(L.T, Q)))
        lam.append(_gpu(lv))
        del m, w, L, S, Q
    for d in range(3):  # V^T M g
        m = _gpu(_axis(c, _dims(c)[d])[0])
        g = _along(V[d].T @ m, g, d)
    g /= 1.0 + lam[2][:, None, None] + lam[1][:, None] + lam[0]
    for d in range(3):
        g = _along(V[d], g, d)
    return g


def _exact_varcoef(c, u, dif, mu):
    """Cell-wise Gauss quadrature with dense point matrices, a few z-cells at a time."""
    p = c["degree"]
    h, _ = _spacing(c)
    per = c["bc"] == "periodic"
    g, w = np.polynomial.legendre.leggauss((3 * p + 2) // 2)
    g, w = 0.5 * (1 + g), 0.5 * w
    axes = []
    for n in _dims(c):
        # one row per point of the cells that meet the index box; cell j spans [j, j+1] (odd) or
        # [j - 1/2, j + 1/2] (even) in units of the spacing, its splines are j - p//2 .. j - p//2 + p
        cells = np.arange(n) if per else np.arange(-(p - p // 2), n + p // 2)
        P, D, E = (np.zeros((len(cells) * len(g), n)) for _ in range(3))
        for t in range(p + 1):
            k = cells - p // 2 + t
            v, dv = _bspline(p, g + 0.5 * (p - 1) - t), _dbspline(p, g + 0.5 * (p - 1) - t)
            for q in range(len(g)):
                rows = np.arange(len(cells)) * len(g) + q
                ok = np.ones(len(k), bool) if per else (k >= 0) & (k < n)
                np.add.at(P, (rows[ok], k[ok] % n), v[q])
                np.add.at(D, (rows[ok], k[ok] % n), dv[q])
                np.add.at(E, (rows, k % n if per else np.clip(k, 0, n - 1)), v[q])
        axes.append((_gpu(P), _gpu(D), _gpu(E), _gpu(np.tile(w, len(cells)))))
    (Px, Dx, Ex, wx), (Py, Dy, Ey, wy), (Pz, Dz, Ez, wz) = axes
    out = torch.zeros_like(u)
    step = max(1, int(3e7) // (Px.shape[0] * Py.shape[0]))
    for a in range(0, Pz.shape[0], step):
        b = slice(a, min(a + step, Pz.shape[0]))
        cv, cz = _along(Pz[b], u, 2), _along(Dz[b], u, 2)
        cvy = _along(Py, cv, 1)
        ww = wz[b][:, None, None] * wy[:, None] * wx
        m = _along(Ex, _along(Ey, _along(Ez[b], mu, 2), 1), 0)
        gv = _along(Px, cvy, 0) * m * ww
        m = _along(Ex, _along(Ey, _along(Ez[b], dif, 2), 1), 0) * ww / h ** 2
        gx = _along(Dx, cvy, 0) * m
        gy = _along(Px, _along(Dy, cv, 1), 0) * m
        gz = _along(Px, _along(Py, cz, 1), 0) * m
        t = _along(Py.T, _along(Px.T, gv, 0) + _along(Dx.T, gx, 0), 1) + _along(Dy.T, _along(Px.T, gy, 0), 1)
        out += _along(Pz[b].T, t, 2) + _along(Dz[b].T, _along(Py.T, _along(Px.T, gz, 0), 1), 2)
    return out


def _conv(x, w, b, per):
    """3x3x3 convolution of x[z][y][x][ci] with w[co][ci][3][3][3]."""
    out = b.expand(*x.shape[:3], len(b)).clone()
    for t in range(27):
        k = (t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1)
        v = x
        for d in range(3):
            if k[d]:
                v = _ShiftFn.apply(v, d, k[d], per)
        out = out + v @ w[:, :, t // 9, t // 3 % 3, t % 3].T
    return out


class _ShiftFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, a, d, k, per):
        ctx.args = d, k, per
        return _shift(a, d, k, per)

    @staticmethod
    def backward(ctx, g):
        d, k, per = ctx.args
        return _shift(g, d, -k, per), None, None, None


def _network(u, q, params, per):
    """The network's output before its scale, from FP64 fields; params: [(W, b)] of the four layers."""
    a = [f / f.square().mean().sqrt() if bool(f.any()) else f for f in (u, q)]
    x = torch.stack(a, -1)
    for i, (w, b) in enumerate(params):
        x = _conv(x, w, b, per)
        if i < 3:
            x = torch.nn.functional.gelu(x)
    o = x[..., 0]
    for _ in range(2):  # the output's binomial low-pass
        for d in (2, 1, 0):
            o = 0.5 * o + 0.25 * (_ShiftFn.apply(o, d, 1, per) + _ShiftFn.apply(o, d, -1, per))
    return o


def _exact_net(c, x):
    w, scale = _weights()
    flat = torch.from_numpy(w).double().to(DEV).requires_grad_(c["kind"] == "net_train")
    params, at = [], 0
    for ci, co in PARAMS:
        params.append((flat[at:at + 27 * ci * co].view(co, ci, 3, 3, 3), flat[at + 27 * ci * co:at + 27 * ci * co + co]))
        at += 27 * ci * co + co
    per = c["bc"] == "periodic"
    tau = _spacing(c)[1]
    if c["kind"] == "net_forward":
        u, q = (t.double() for t in x)
        return _network(u, q, params, per) * (tau * scale * u.square().mean().sqrt())
    loss = 0.0
    for u, q, du in zip(*x):
        u, q, du = u.double(), q.double(), du.double()
        o = _network(u, q, params, per)
        part = (o - du / (tau * scale * u.square().mean().sqrt())).square().mean() / c["batch"]
        part.backward()
        loss += float(part.detach())
    return {"loss": loss, "grad": flat.grad}


def exact(case, seed):
    c = dict(case)
    x = _inputs(c, seed)
    kind = c["kind"]
    if kind == "step":
        return _exact_step(c, *x)
    if kind == "apply":
        return _exact_apply(c, x[0].double())
    if kind == "varcoef":
        return _exact_varcoef(c, *(t.double() for t in x))
    if kind == "transform":
        taps = [_bspline(c["degree"], float(k)) for k in range(c["degree"] // 2 + 1)]
        coef = x[0].clone()
        for d, n in enumerate(_dims(c)):
            coef = _along(_gpu(np.linalg.inv(_band(taps, n, c["bc"]))), coef, d)
        return {"coef": coef, "samples": x[0]}
    return _exact_net(c, x)
