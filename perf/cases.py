"""Performance cases of the framework: what its users have it compute.

Six solves (GMRES on the 2D FDFD operator, alone and in lockstep batches, plain
and augmented), the convolutional predictor's inference and its gradient, and
the three preparatory computations of the predictors (principal components,
local training targets, effective-index fields).  Every case goes through the
public Python entry points of the package.

Solves run to a true relative residual at which the field is converged, and the
fields are returned in complex64, the type in which the library's own training
and recycling code keeps solved fields.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1902_00090_amd import (Cnn, FdfdOp, Solver, eim_field, gmres_solve_batched,
                                  local_pca_targets, pca_build)

EPS_LO, EPS_HI = 2.085, 12.25          # silica, silicon
DX = 0.025                             # um per cell
DEV = "cuda"


# --------------------------------------------------------------------- cases ----
def listed():
    return [
        # one small random-pixel device solved in double precision with the
        # library's default two Gram-Schmidt passes: the smallest solve, bound
        # by latency
        dict(name="solve small c128", kind="solve", shape="binary", nx=64, ny=64, npml=10, batch=1,
             k=0, inner="c128", passes=2, restart=50, tol=1e-8, graph=False, fused=False),
        # one full-size grating alone, step groups replayed as graphs
        dict(name="solve one grating", kind="solve", shape="grating", nx=480, ny=240, npml=20,
             batch=1, k=0, inner="c64", passes=1, restart=100, tol=1e-7, graph=True, fused=False),
        # one mid-size grating augmented by predicted fields, one sweep per step
        dict(name="solve one augmented", kind="solve", shape="grating", nx=320, ny=160, npml=20,
             batch=1, k=10, inner="c64", passes=1, restart=100, tol=1e-7, graph=False, fused=True),
        # a batch of small gratings in lockstep: snapshots for the predictors
        dict(name="solve batch 48", kind="solve", shape="grating", nx=192, ny=96, npml=20,
             batch=48, k=0, inner="c64", passes=1, restart=100, tol=1e-7, graph=False, fused=False),
        # a batch of test devices augmented by a predicted subspace
        dict(name="solve batch augmented", kind="solve", shape="grating", nx=256, ny=128, npml=20,
             batch=20, k=20, inner="c64", passes=1, restart=100, tol=1e-7, graph=False,
             fused=False),
        # devices of three sizes, one an odd one, in one lockstep batch, through
        # the one-call solver with its default options
        dict(name="solve uneven default", kind="uneven", grids="192x96,160x80,251x117", batch=9,
             npml=20, restart=100, tol=1e-7),
        # a subspace for one new device, as a serving loop asks for it
        dict(name="cnn predict one", kind="predict", nx=480, ny=240, batch=1, k=10, planes=3),
        # subspaces for a batch of new devices
        dict(name="cnn predict batch", kind="predict", nx=480, ny=240, batch=64, k=10, planes=3),
        # forward and backward of one training batch
        dict(name="cnn gradient", kind="grad", nx=480, ny=240, batch=32, k=10, planes=3),
        # principal components of solved fields
        dict(name="pca", kind="pca", nx=480, ny=240, fields=1000, k=20),
        # training targets of the fields of one design trajectory
        dict(name="targets", kind="targets", nx=480, ny=240, fields=32, window=8, k=10),
        # effective-index fields of a batch: the predictor's second input
        dict(name="effective index", kind="eim", nx=480, ny=240, npml=20, batch=64),
    ]


def _iterations(nx, ny):
    """Arnoldi steps that GMRES(100) typically takes on a grating of this size."""
    return 0.72 * (nx * ny) ** 0.83


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "uneven", "predict", "grad", "pca", "targets",
                       "eim"])
    nx4, ny4 = 4 * _log(rng, 16, 120), 4 * _log(rng, 12, 60)
    nx, ny = _log(rng, 96, 480), _log(rng, 72, 240)
    npml = rng.randint(10, 20)
    if kind == "solve":
        if rng.random() < 0.2:
            n = rng.randint(48, 72)
            return dict(kind="solve", shape="binary", nx=n, ny=n + rng.randint(-6, 6), npml=10,
                        batch=1, k=0, inner="c128", passes=rng.choice([1, 2]),
                        restart=rng.randint(40, 60), tol=1e-8, graph=rng.random() < 0.3,
                        fused=False)
        k, passes = rng.choice([0, 0, rng.randint(1, 20)]), rng.choice([1, 1, 2])
        # cells x iterations x basis no more than those of the listed batches
        most = 48 * 192 * 96 * _iterations(192, 96) / (nx * ny * _iterations(nx, ny))
        most = max(1, int(most / passes * 50 / (50 + k)))
        batch = 1 if rng.random() < 0.3 else min(most, _log(rng, 2, 64))
        return dict(kind="solve", shape="grating", nx=nx, ny=ny, npml=npml, batch=batch, k=k,
                    inner="c64", passes=passes, restart=rng.choice([80, 100]), tol=1e-7,
                    graph=rng.random() < 0.3, fused=rng.random() < 0.2)
    if kind == "uneven":
        grids = ",".join("%dx%d" % (_log(rng, 96, 256), _log(rng, 72, 120)) for _ in range(3))
        return dict(kind="uneven", grids=grids, batch=rng.randint(3, 9), npml=npml, restart=100,
                    tol=1e-7)
    if kind == "predict":
        return dict(kind="predict", nx=nx4, ny=ny4, batch=_log(rng, 1, 64), k=rng.randint(4, 16),
                    planes=rng.choice([1, 3]))
    if kind == "grad":
        return dict(kind="grad", nx=nx4, ny=ny4, batch=_log(rng, 2, 32), k=rng.randint(4, 10),
                    planes=rng.choice([1, 3]))
    if kind == "pca":
        return dict(kind="pca", nx=nx, ny=ny, fields=_log(rng, 64, 1000), k=rng.randint(5, 20))
    if kind == "targets":
        return dict(kind="targets", nx=nx, ny=ny, fields=rng.randint(8, 32),
                    window=rng.randint(4, 8), k=rng.randint(4, 10))
    return dict(kind="eim", nx=nx, ny=ny, npml=npml, batch=_log(rng, 1, 64))


# ------------------------------------------------------------------- devices ----
def _smooth(rng, ny, nx, sigma=3.0):
    """Normal noise under a Gaussian filter (periodic), standardised."""
    z = np.fft.rfft2(rng.standard_normal((ny, nx)))
    fy, fx = np.fft.fftfreq(ny)[:, None], np.fft.rfftfreq(nx)[None]
    z = np.fft.irfft2(z * np.exp(-2 * (math.pi * sigma) ** 2 * (fx ** 2 + fy ** 2)), (ny, nx))
    return (z - z.mean()) / z.std()


@functools.lru_cache(maxsize=64)
def _slab_mode(ny, omega):
    """Fundamental mode of the column through the input waveguide, peak 1."""
    e = np.full(ny, EPS_LO)
    e[ny // 2 - 8:ny // 2 + 8] = EPS_HI
    T = np.diag(omega ** 2 * e - 2 / DX ** 2)
    i = np.arange(ny - 1)
    T[i, i + 1] = T[i + 1, i] = 1 / DX ** 2
    u = np.linalg.eigh(T)[1][:, -1]
    return u / u[np.argmax(np.abs(u))]


def _device(rng, shape, nx, ny, npml):
    """(eps float32 [ny, nx], b complex128 [ny*nx], omega, dx) of one device."""
    J = np.zeros((ny, nx))
    if shape == "binary":
        omega, dx = 2 * math.pi / 1.55, 0.040
        eps = np.full((ny, nx), EPS_LO)
        y0, x0 = ny // 4, nx // 4
        pix = rng.random((ny - 2 * y0, nx - 2 * x0)) < 0.5
        eps[y0:ny - y0, x0:nx - x0] = np.where(pix, EPS_HI, EPS_LO)
        J[:, npml + 2] = 1.0
    else:
        omega, dx = 2 * math.pi / rng.choice([1.30, 1.55]), DX
        eps = np.full((ny, nx), EPS_LO)
        wx, wy = int(round(5 * nx / 12)), ny // 3
        x0, y0 = (nx - wx) // 2, (ny - wy) // 2
        eps[ny // 2 - 8:ny // 2 + 8] = EPS_HI
        eps[y0:y0 + wy, x0:x0 + wx] = EPS_LO + (EPS_HI - EPS_LO) / (
            1 + np.exp(-2 * _smooth(rng, wy, wx)))
        J[:, npml + 10] = _slab_mode(ny, omega)
    return eps.astype(np.float32), (-1j * omega * J).reshape(-1), omega, dx


def _grids(case):
    if case["kind"] == "uneven":
        g = [tuple(int(v) for v in s.split("x")) for s in case["grids"].split(",")]
        return [g[p % len(g)] for p in range(case["batch"])]
    return [(case["nx"], case["ny"])] * case["batch"]


def _devices(case, seed):
    rng = np.random.default_rng(seed)
    return [_device(rng, case.get("shape", "grating"), nx, ny, case["npml"])
            for nx, ny in _grids(case)]


def _weights(case, seed):
    """Flat network parameters, He-uniform with small biases, as in training."""
    rng = np.random.default_rng(seed)
    out = []
    for cin, cout, _, _, _ in _layers(case):
        h = math.sqrt(6 / (9 * cin))
        out += [rng.uniform(-h, h, cout * cin * 9), rng.uniform(-0.05, 0.05, cout)]
    return np.concatenate(out).astype(np.float32)


def _layers(case):
    k, c = case["k"], case["planes"]
    return [(c, 32, 1, 0, 1), (32, 64, 2, 0, 1), (64, 128, 2, 0, 1), (128, 128, 1, 0, 1),
            (128, 64, 1, 1, 1), (64, 32, 1, 1, 1), (32, 32, 1, 0, 1), (32, 2 * k, 1, 0, 0)]


def _waves(g, n, nx, ny):
    """n unit-RMS complex fields [n, ny*nx]: a few plane waves each."""
    x = torch.arange(nx, device=DEV, dtype=torch.float32)
    y = torch.arange(ny, device=DEV, dtype=torch.float32)
    q = torch.rand((n, 6, 4), device=DEV, generator=g)
    kx, ky, ph = q[..., 0] * 0.4, (q[..., 1] - 0.5) * 0.4, q[..., 2] * 2 * math.pi
    a = torch.exp(1j * (kx[..., None] * x + ph[..., None])) * q[..., 3:]
    F = torch.einsum("nax,nay->nyx", a, torch.exp(1j * ky[..., None] * y)).reshape(n, ny * nx)
    return (F / F.abs().square().mean(1, keepdim=True).sqrt()).contiguous()


def _images(case, seed):
    """(eps [B, ny, nx], eim [B, D] or None, targets [B, k, D]) on the GPU."""
    B, nx, ny = case["batch"], case["nx"], case["ny"]
    g = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    eps = np.full((B, ny, nx), EPS_LO, np.float32)
    wx, wy = int(round(5 * nx / 12)), ny // 3
    x0, y0 = (nx - wx) // 2, (ny - wy) // 2
    eps[:, ny // 2 - 8:ny // 2 + 8] = EPS_HI
    for e in eps:
        e[y0:y0 + wy, x0:x0 + wx] = EPS_LO + (EPS_HI - EPS_LO) / (
            1 + np.exp(-2 * _smooth(rng, wy, wx)))
    eim = _waves(g, B, nx, ny) if case["planes"] == 3 else None
    t = None
    if case["kind"] == "grad":
        t = _waves(g, B * case["k"], nx, ny).reshape(B, case["k"], nx * ny)
    return torch.tensor(eps, device=DEV), eim, t


def _fields(case, seed):
    """Fields of a decaying spectrum: combinations of common patterns, each with
    a part of its own, as the solutions of related devices have."""
    n, nx, ny = case["fields"], case["nx"], case["ny"]
    g = torch.Generator(device=DEV).manual_seed(seed)
    m = 40
    base = _waves(g, m, nx, ny) * (0.85 ** torch.arange(m, device=DEV))[:, None]
    mix = torch.randn((n, m), device=DEV, generator=g, dtype=torch.complex64)
    F = mix @ base
    for c in range(0, n, 100):
        own = torch.randn((min(100, n - c), nx * ny), device=DEV, generator=g,
                          dtype=torch.complex64)
        F[c:c + 100] += 0.05 * own
    return F


# ----------------------------------------------------------------- the cases ----
def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("solve", "uneven", "eim"):
        dev = _devices(case, seed)
        s["ops"] = [FdfdOp(e, om, dx, case["npml"]) for e, _, om, dx in dev]
        s["b"] = [torch.tensor(b, dtype=torch.complex128, device=DEV) for _, b, _, _ in dev]
    if kind == "solve":
        s["solver"] = Solver(s["ops"], restart=case["restart"], kmax=case["k"], inner=case["inner"],
                             cgs_passes=case["passes"], use_graph=case["graph"],
                             fused=case["fused"])
        s["U"] = None
        if case["k"]:
            # the fields of a cheap model on k other devices of the same kind
            other = _devices(dict(case, batch=case["k"]), seed + 1_000_003)
            ops = [FdfdOp(e, om, dx, case["npml"]) for e, _, om, dx in other]
            b = [torch.tensor(v, dtype=torch.complex128, device=DEV) for _, v, _, _ in other]
            s["U"] = [torch.stack(eim_field(ops, b))] * case["batch"]
    elif kind in ("predict", "grad"):
        s["net"] = Cnn(case["nx"], case["ny"], case["batch"], k=case["k"],
                       in_channels=case["planes"])
        s["net"].set_params(_weights(case, seed))
        s["eps"], s["eim"], s["target"] = _images(case, seed)
    elif kind in ("pca", "targets"):
        s["F"] = _fields(case, seed)
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "solve":
        if s["U"] is not None:
            s["solver"].set_subspace(s["U"])
        x, _, _ = s["solver"].solve(s["b"], tol=c["tol"], maxit=60000)
        return torch.stack(x).to(torch.complex64)
    if kind == "uneven":
        x, _, _ = gmres_solve_batched(s["ops"], s["b"], tol=c["tol"], restart=c["restart"],
                                      maxit=60000)
        return torch.cat(x).to(torch.complex64)
    if kind == "predict":
        return s["net"].predict(s["eps"], eim=s["eim"])
    if kind == "grad":
        loss, grad = s["net"].grad(s["eps"], s["target"], eim=s["eim"])
        return {"loss": loss, "grad": grad}
    if kind == "pca":
        U, sigma = pca_build(s["F"], c["k"])
        return {"U": U, "sigma": sigma}
    if kind == "targets":
        return local_pca_targets(s["F"], c["window"], c["k"])
    return torch.stack(eim_field(s["ops"], s["b"]))


def work(case):
    kind = case["kind"]
    if kind in ("solve", "uneven"):
        # restarted GMRES: every Arnoldi step reads the basis that there is once
        # and writes one vector; 16 flops a basis value (dots and update).  The
        # number of steps is the typical one of the grid's size.
        size = 16 if case.get("inner") == "c128" else 8
        m, k = case["restart"], case.get("k", 0)
        cells = 0.0
        for nx, ny in _grids(case):
            its = 2400 if case.get("shape") == "binary" else _iterations(nx, ny)
            cells += its * nx * ny
        return {"bytes": cells * size * (k + m / 2 + 3), "flops": cells * 16 * (k + m / 2)}
    D = case["nx"] * case["ny"]
    if kind in ("predict", "grad"):
        H, W, flops = case["ny"], case["nx"], 0
        act = 0                                  # layer outputs, 2 bytes a value
        for cin, cout, s, up, _ in _layers(case):
            H, W = (2 * H, 2 * W) if up else (H // s, W // s)
            flops += 18 * cin * cout * H * W
            act += 2 * cout * H * W
        B, io = case["batch"], D * (4 + 8 * (case["planes"] == 3) + 8 * case["k"])
        if kind == "predict":
            return {"bytes": B * io, "flops": B * flops}
        # the backward pass reads every layer's output again
        return {"bytes": B * (io + 2 * act), "flops": 3 * B * flops}
    if kind == "pca":
        M = case["fields"]
        return {"bytes": 8 * D * (M + case["k"]), "flops": 8 * D * (M * (M + 1) / 2 + M * case["k"])}
    if kind == "targets":
        S, k = case["fields"], case["k"]
        near = min(S, 2 * case["window"] + 1)
        return {"bytes": 8 * D * S * (1 + k), "flops": 8 * D * (S * (S + 1) / 2 + S * near * k)}
    # the permittivity read, the field written; bisection and inverse iteration
    return {"bytes": case["batch"] * D * (8 + 8), "flops": case["batch"] * D * 4 * 60}


# --------------------------------------------------------------- in 64 bits ----
def _stretch(n, npml, dx, omega):
    def s(p):
        d = np.minimum(np.maximum(0, np.maximum(npml - p, p - (n - 1 - npml))), npml)
        return 1 - 1j * (4 * 16.0 / (2 * npml * dx)) * (d / npml) ** 3 / omega
    i = np.arange(n, dtype=np.float64)
    return s(i), s(i + 0.5)


def _axis(n, npml, dx, omega):
    """Couplings (down, up) of node i to i - 1 and i + 1."""
    si, sh = _stretch(n, npml, dx, omega)
    return 1 / (dx * dx * si * np.roll(sh, 1)), 1 / (dx * dx * si * sh)


def _solve64(dev, npml):
    """Fields of devices of one grid, directly: block elimination along x with
    the last column as the separator of the periodic wrap."""
    ny, nx = dev[0][0].shape
    z = torch.complex128

    def put(a):
        return torch.tensor(np.stack(a), dtype=z, device=DEV)

    cx = [_axis(nx, npml, dx, om) for _, _, om, dx in dev]
    cy = [_axis(ny, npml, dx, om) for _, _, om, dx in dev]
    dn, up = put([c[0] for c in cx]), put([c[1] for c in cx])              # [B, nx]
    yd, yu = put([c[0] for c in cy]), put([c[1] for c in cy])              # [B, ny]
    w2 = torch.tensor([om * om for _, _, om, _ in dev], device=DEV)
    eps = torch.tensor(np.stack([e for e, _, _, _ in dev]), dtype=torch.float64, device=DEV)
    b = put([v.reshape(ny, nx) for _, v, _, _ in dev])
    B, r = len(dev), torch.arange(ny, device=DEV)
    Y = torch.zeros((B, ny, ny), dtype=z, device=DEV)
    Y[:, r, r] += yd + yu
    Y[:, r, (r - 1) % ny] -= yd
    Y[:, r, (r + 1) % ny] -= yu

    def column(i):
        T = Y.clone()
        T[:, r, r] += (dn[:, i] + up[:, i])[:, None] - w2[:, None] * eps[:, :, i]
        return T

    eye = torch.eye(ny, dtype=z, device=DEV).expand(B, ny, ny)
    # columns 0 .. nx - 2: right-hand sides [b | coupling to column nx - 1]
    inv, rhs = [], []
    for i in range(nx - 1):
        S = column(i)
        R = torch.cat([b[:, :, i:i + 1], torch.zeros_like(eye)], 2)
        if i == 0:
            R[:, :, 1:] += dn[:, 0, None, None] * eye
        if i == nx - 2:
            R[:, :, 1:] += up[:, i, None, None] * eye
        if i > 0:
            S = S - (dn[:, i] * up[:, i - 1])[:, None, None] * inv[-1]
            R = R + dn[:, i, None, None] * torch.bmm(inv[-1], rhs[-1])
        inv.append(torch.linalg.inv(S))
        rhs.append(R)
    sol = [None] * (nx - 1)
    for i in range(nx - 2, -1, -1):
        R = rhs[i] if i == nx - 2 else rhs[i] + up[:, i, None, None] * sol[i + 1]
        sol[i] = torch.bmm(inv[i], R)
        rhs[i] = inv[i] = None
    last = nx - 1
    u, d = up[:, last, None, None], dn[:, last, None, None]
    S = column(last) - u * sol[0][:, :, 1:] - d * sol[-1][:, :, 1:]
    x = b[:, :, last:] + u * sol[0][:, :, :1] + d * sol[-1][:, :, :1]
    x = torch.linalg.solve(S, x)
    cols = [s[:, :, :1] + torch.bmm(s[:, :, 1:], x) for s in sol] + [x]
    return torch.cat(cols, 2).reshape(B, ny * nx)


def _eim64(dev, npml):
    """Effective-index fields: the lowest mode of every column by bisection and
    inverse iteration, then the line equation along x."""
    ny, nx = dev[0][0].shape
    B = len(dev)
    om = torch.tensor([d[2] for d in dev], dtype=torch.float64, device=DEV)
    dx = dev[0][3]
    eps = torch.tensor(np.stack([d[0] for d in dev]), dtype=torch.float64, device=DEV)
    diag = (2 / dx ** 2 - om[:, None, None] ** 2 * eps).permute(1, 0, 2).reshape(ny, B * nx)
    off = 1 / dx ** 2
    lo, hi = diag.min(0)[0] - 2 * off, diag.min(0)[0] + 2 * off
    for _ in range(70):
        mid = (lo + hi) / 2
        q = diag[0] - mid
        neg = q < 0
        for i in range(1, ny):
            q = diag[i] - mid - off * off / q
            neg = neg | (q < 0)
        lo, hi = torch.where(neg, lo, mid), torch.where(neg, mid, hi)
    # just below the eigenvalue the shifted matrix is positive definite
    mu, shift = (lo + hi) / 2, lo - 1e-9 * lo.abs() - 1e-9
    v = torch.ones_like(diag)
    for _ in range(4):
        c, y = [None] * ny, [None] * ny
        for i in range(ny):
            p = diag[i] - shift - (off * c[i - 1] if i else 0)
            c[i] = off / p
            y[i] = (v[i] + (off * y[i - 1] if i else 0)) / p
        for i in range(ny - 2, -1, -1):
            y[i] = y[i] + c[i] * y[i + 1]
        v = torch.stack(y)
        v = v / v.norm(dim=0)
    phi = v.reshape(ny, B, nx).permute(1, 0, 2)
    b = torch.tensor(np.stack([d[1].reshape(ny, nx) for d in dev]), device=DEV)
    j = (phi * b).sum(1)
    cx = [_axis(nx, npml, d[3], d[2]) for d in dev]
    dn = torch.tensor(np.stack([c[0] for c in cx]), device=DEV)
    up = torch.tensor(np.stack([c[1] for c in cx]), device=DEV)
    r = torch.arange(nx, device=DEV)
    A = torch.zeros((B, nx, nx), dtype=torch.complex128, device=DEV)
    A[:, r, r] += dn + up + mu.reshape(B, nx)
    A[:, r, (r - 1) % nx] -= dn
    A[:, r, (r + 1) % nx] -= up
    a = torch.linalg.solve(A.cpu(), j.cpu()).to(DEV)
    return (phi * a[:, None]).reshape(B, ny * nx)


def _net64(case, params, eps, eim):
    """The network on one image, channels first, in 64 bits (differentiable)."""
    ny, nx = case["ny"], case["nx"]
    x = ((eps.double() - EPS_LO) / (EPS_HI - EPS_LO))[None]
    if eim is not None:
        f = eim.to(torch.complex128)
        f = (f / f.abs().square().mean().sqrt()).reshape(ny, nx)
        x = torch.cat([x, f.real[None], f.imag[None]])
    for (cin, cout, s, up, relu), (w, bias) in zip(_layers(case), params):
        if up:
            x = x.repeat_interleave(2, 1).repeat_interleave(2, 2)
        H, W = x.shape[1:]
        xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
        y = bias[:, None]
        for dy in range(3):
            for dx in range(3):
                part = xp[:, dy:dy + H:s, dx:dx + W:s]
                y = y + w[:, :, dy, dx] @ part.reshape(cin, -1)
        x = y.reshape(cout, H // s, W // s)
        if relu:
            x = x.relu()
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "uneven"):
        dev = _devices(case, seed)
        out = [None] * len(dev)
        for g in set(_grids(case)):
            at = [p for p, h in enumerate(_grids(case)) if h == g]
            for c in range(0, len(at), 8):
                for p, x in zip(at[c:c + 8], _solve64([dev[p] for p in at[c:c + 8]], case["npml"])):
                    out[p] = x
        return torch.stack(out) if kind == "solve" else torch.cat(out)
    if kind in ("predict", "grad"):
        eps, eim, target = _images(case, seed)
        flat = torch.tensor(_weights(case, seed), dtype=torch.float64, device=DEV)
        flat.requires_grad_(kind == "grad")
        params, at = [], 0
        for cin, cout, _, _, _ in _layers(case):
            n = cout * cin * 9
            params.append((flat[at:at + n].reshape(cout, cin, 3, 3), flat[at + n:at + n + cout]))
            at += n + cout
        outs, loss = [], 0.0
        for i in range(case["batch"]):
            y = _net64(case, params, eps[i], None if eim is None else eim[i])
            if kind == "predict":
                f = torch.complex(y[0::2], y[1::2]).reshape(case["k"], -1)
                outs.append(f)
                continue
            t = target[i].reshape(case["k"], case["ny"], case["nx"]).to(torch.complex128)
            t = torch.stack([t.real, t.imag], 1).reshape(y.shape)
            part = (y - t).square().mean() / case["batch"]
            part.backward()
            loss += float(part.detach())
        if kind == "predict":
            return torch.stack(outs)
        return {"loss": loss, "grad": flat.grad}
    if kind == "pca":
        F = _fields(case, seed).to(torch.complex128)
        G = (F @ F.conj().T.contiguous()).cpu()
        s = torch.linalg.eigvalsh(G).flip(0)[:case["k"]].sqrt()
        return {"U": None, "sigma": s}           # a singular vector's phase is free
    if kind == "targets":
        F = _fields(case, seed).to(torch.complex128)
        F = F / F.norm(dim=1, keepdim=True)
        S, k = len(F), case["k"]
        out = torch.zeros((S, k, F.shape[1]), dtype=torch.complex128, device=DEV)
        for s in range(S):
            part = F[max(0, s - case["window"]):s + case["window"] + 1]
            G = (part.conj() @ part.T.contiguous()).cpu()
            w, V = torch.linalg.eigh(G)
            kk = min(k, len(part))
            w, V = w.flip(0)[:kk].to(DEV), V.flip(1)[:, :kk].to(DEV)
            u = (V / w.sqrt()).T.contiguous() @ part
            out[s, :kk] = u * (u.conj() @ F[s])[:, None]
        return out
    return _eim64(_devices(case, seed), case["npml"])
