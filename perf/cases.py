"""The workloads by which this framework's speed is followed.

Each case is one pass through a public entry point, on inputs made from a seed:

  op         ``Cisor.apply_A``: the Lippmann-Schwinger operator A or A^H on every
             transmitter's field (2D and 3D; what a caller's own solver loops over)
  forward    ``Cisor.forward``: fields and receiver data of a known contrast
  grad       ``Cisor.grad``: misfit, fields and Prop. 1 gradient, the body of every
             reconstruction step
  data       ``Cisor.project`` with measured data and ``Cisor.backproject`` of the
             residual: the receiver contractions by themselves
  tv         ``Cisor.tv_prox``: the TV/box proximal step (2D and 3D)
  vec        ``VecCisor.grad``: the gradient of the 3D vectorial model
  predict    ``WarmStartNet.predict``: the learned starting fields
  train      ``WarmStartNet.loss_grad``: the network's loss and parameter gradient

Not here: the grouped batch (``Batch``), whose full recipe is disabled.

``exact`` computes the same outputs in 64 bits with torch alone, from the
formulas of the model (cell-integrated Green's functions, FFT convolution,
BiCGSTAB to 1e-12, FGP).
"""

from __future__ import annotations

import math

import numpy as np
import torch

DEV = "cuda"
INNER = 100            # FGP iterations of the proximal step
TV_LAM = 0.02


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest call: a 32^2 complex128 problem's adjoint operator, all launch latency
        dict(name="op_32x8_c128_adj", kind="op", dim=2, n=32, T=8, prec="c128", adj=True),
        # the operator of the headline reconstruction, 256^2 pixels and 60 transmitters
        dict(name="op_256x60", kind="op", dim=2, n=256, T=60, prec="c64", adj=False),
        # the operator of the 3D scalar reconstruction, 64^3 voxels and 16 transmitters
        dict(name="op3d_64x16", kind="op", dim=3, n=64, T=16, prec="c64", adj=False),
        # the small complex128 configuration's forward model, solved to 1e-8
        dict(name="forward_32x8_c128", kind="forward", n=32, T=8, M=32, prec="c128", tol=1e-8, eps=1.5),
        # fields and data of a mid-size object on an odd grid, 25 sources, 338 receivers
        dict(name="forward_125x25", kind="forward", n=125, T=25, M=338, prec="c64", tol=1e-6, eps=1.3),
        # the body of a headline reconstruction step: 60 transmitters, 360 receivers
        dict(name="grad_256x60", kind="grad", n=256, T=60, M=360, prec="c64", tol=1e-6, eps=1.1),
        # the receiver contractions of the headline problem
        dict(name="data_256x60x360", kind="data", n=256, T=60, M=360, prec="c64"),
        # the proximal step of the headline problem
        dict(name="tv_256", kind="tv", dim=2, n=256, prec="c64"),
        # the proximal step of the 3D scalar reconstruction
        dict(name="tv3d_64", kind="tv", dim=3, n=64, prec="c64"),
        # the vectorial gradient on the 3D experimental layout's size
        dict(name="vec_32x81", kind="vec", n=32, T=81, M=36, tol=1e-6, eps=1.3),
        # starting fields for 16 transmitters from the trained network
        dict(name="predict_128x16", kind="predict", n=128, B=16),
        # the body of a training step, a batch of 16 fields
        dict(name="train_128x16", kind="train", n=128, B=16),
    ]


def draw(rng):
    """One more case of the same ranges (sizes log-uniform, odd ones among them)."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["op", "op", "op3d", "forward", "forward", "grad", "grad", "data", "data", "tv", "tv3d", "vec",
                       "predict", "train"])
    prec = "c128" if rng.random() < 0.3 else "c64"
    if kind == "op":
        n = size(24, 512)
        return dict(kind="op", dim=2, n=n, T=max(1, min(size(4, 64), 60 * 256 ** 2 // n ** 2)), prec=prec,
                    adj=rng.random() < 0.5)
    if kind == "op3d":
        return dict(kind="op", dim=3, n=size(14, 56), T=size(2, 16), prec=prec, adj=rng.random() < 0.5)
    if kind == "forward":
        n = size(24, 200)
        return dict(kind="forward", n=n, T=size(4, 40), M=size(24, 360), prec=prec,
                    tol=1e-8 if prec == "c128" else 1e-6, eps=round(rng.uniform(1.1, 1.4), 2))
    if kind == "grad":
        n = size(32, 240)
        return dict(kind="grad", n=n, T=size(4, 40), M=size(32, 338), prec=prec,
                    tol=1e-8 if prec == "c128" else 1e-6, eps=round(rng.uniform(1.05, 1.2), 2))
    if kind == "data":
        return dict(kind="data", n=size(32, 240), T=size(4, 80), M=size(32, 360), prec=prec)
    if kind == "tv":
        return dict(kind="tv", dim=2, n=size(24, 512), prec=prec)
    if kind == "tv3d":
        return dict(kind="tv", dim=3, n=size(12, 63), prec=prec)
    if kind == "vec":
        return dict(kind="vec", n=size(10, 31), T=size(6, 80), M=size(12, 36), tol=1e-6,
                    eps=round(rng.uniform(1.1, 1.4), 2))
    n = rng.choice([64, 96, 128])      # a batch's pixels are a multiple of 8192
    return dict(kind=kind, n=n, B=8 * rng.randint(1, 2) if n == 96 else 2 * rng.randint(1, 8))


# ---------------------------------------------------------------- geometry and inputs
def pixel(case):
    """Pixel side in wavelengths."""
    return 1.0 / 6 if case.get("dim") == 3 else (4.7 / 74.9 if case["kind"] == "vec" else 0.1)


def ring(M, radius):
    ph = 2 * np.pi * np.arange(M) / M
    return radius * np.stack([np.cos(ph), np.sin(ph)], 1)


def directions(case):
    T = case.get("T", case.get("B", 1))
    a = 2 * np.pi * np.arange(T) / T
    if case.get("dim") == 3:       # a downward cone of 45 degrees
        return np.stack([np.cos(a), np.sin(a), -np.ones(T)], 1) / math.sqrt(2.0)
    if case["kind"] == "vec":      # a spiral over the band of polar angles 30..150 degrees
        th = np.deg2rad(30.0 + 120.0 * (np.arange(T) + 0.5) / T)
        ph = 2.399963 * np.arange(T)
        return -np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], 1)
    return np.stack([np.cos(a), np.sin(a)], 1)


def receivers(case):
    n, h = case["n"], pixel(case)
    if case.get("dim") == 3:
        return np.array([[0.0, 0.0, -float(n) * h]])
    if case["kind"] == "vec":
        r = ring(case["M"], 1769.0 / 74.9)
        return np.concatenate([r, np.zeros((case["M"], 1))], 1)
    return ring(case.get("M", 8), n * h)


def phantom(n, dim, seed, top):
    """A large random ellipse (ellipsoid) with smaller ones inside; contrasts up to top - 1."""
    rng = np.random.default_rng(seed)
    x = np.linspace(-1, 1, n)
    g = np.meshgrid(*([x] * dim), indexing="ij")
    f = np.zeros((n,) * dim)
    for i in range(6):
        ax = rng.uniform(0.6, 0.9, dim) if i == 0 else rng.uniform(0.1, 0.35, dim)
        c = np.zeros(dim) if i == 0 else rng.uniform(-0.4, 0.4, dim)
        inside = sum(((gd - cd) / a) ** 2 for gd, cd, a in zip(g, c, ax)) <= 1
        f[inside] = (top - 1.0) * rng.uniform(0.2, 1.0)
    return f


def gaussian(seed, *shape):
    """Standard complex normal values, the same on every machine."""
    rng = np.random.default_rng(seed)
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def real_t(case):
    return torch.float64 if case.get("prec") == "c128" or case["kind"] == "vec" else torch.float32


def cplx_t(case):
    return torch.complex128 if real_t(case) == torch.float64 else torch.complex64


def fields_of(case, seed, rows):
    """A smooth part, as a plane wave has, and a rough one, as a residual has."""
    n, dim = case["n"], case["dim"]
    g = torch.Generator().manual_seed(seed)
    N = n ** dim
    x = torch.view_as_complex(torch.randn(rows, N, 2, generator=g, dtype=torch.float32)).to(torch.complex128)
    ph = 2 * math.pi * pixel(case) * torch.arange(N, dtype=torch.float64).remainder(n)
    return 0.5 * x + torch.polar(torch.ones_like(ph), ph)


def inputs(case, seed):
    """The case's input arrays on the host, in the precision the library takes."""
    k, rt, ct = case["kind"], real_t(case), cplx_t(case)
    n = case["n"]
    as_r = lambda a: torch.as_tensor(np.ascontiguousarray(a)).reshape(-1).to(rt)  # noqa: E731
    if k == "op":
        return dict(f=as_r(phantom(n, case["dim"], seed, 1.5)), x=fields_of(case, seed, case["T"]).to(ct))
    if k == "forward":
        return dict(f=as_r(phantom(n, 2, seed, case["eps"])))
    if k == "grad":
        return dict(f=as_r(phantom(n, 2, seed, case["eps"])),
                    y=torch.as_tensor(0.3 * gaussian(seed, case["T"], case["M"])).to(ct))
    if k == "data":
        return dict(f=as_r(phantom(n, 2, seed, 1.5)), u=fields_of(dict(case, dim=2), seed, case["T"]).to(ct),
                    y=torch.as_tensor(0.3 * gaussian(seed, case["T"], case["M"])).to(ct))
    if k == "tv":
        z = phantom(n, case["dim"], seed, 2.0)
        return dict(z=as_r(z + 0.1 * np.random.default_rng(seed).standard_normal(z.shape)))
    if k == "vec":
        return dict(f=as_r(phantom(n, 3, seed, case["eps"])),
                    y=torch.as_tensor(0.01 * gaussian(seed, case["T"], case["M"])))
    B, N = case["B"], n * n
    f = np.stack([phantom(n, 2, seed + 17 * b, 2.0).reshape(-1) for b in range(B)])
    ax = (np.arange(n) - (n - 1) / 2) * 0.1
    d = directions(case)
    ui = np.exp(2j * np.pi * (d[:, :1, None] * ax[None, :, None] + d[:, 1:, None] * ax[None, None, :]))
    ui = ui.reshape(B, N)
    ub = 0.3 * f * ui * np.exp(0.5j)
    u = ui + ub + 0.05 * gaussian(seed, B, N)
    c = lambda a: torch.as_tensor(a).to(torch.complex64)  # noqa: E731
    return dict(f=torch.as_tensor(f).to(torch.float32), ui=c(ui), ub=c(ub), u=c(u))


_handles: dict = {}


def handle(case):
    """The operator context (or network) of a geometry: a program makes it once and keeps it,
    whatever contrasts and data it then works on.  Only the last one is kept here."""
    key = tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "adj", "tol", "eps")))
    if key in _handles:
        return _handles[key]
    for h in _handles.values():
        h.close()
    _handles.clear()
    if case["kind"] == "vec":
        from paper_1708_01663_amd.vec3d import VecCisor
        op = VecCisor(case["n"], pixel(case), directions(case), receivers(case))
    elif case["kind"] in ("predict", "train"):
        from paper_1708_01663_amd.warmstart import DEFAULT_WEIGHTS, WarmStartNet
        op = WarmStartNet(case["n"], case["n"], 32, max_batch=case["B"])
        op.set_params(np.load(DEFAULT_WEIGHTS, allow_pickle=False)["params"])
    else:
        from paper_1708_01663_amd.cisor import Cisor
        op = Cisor(case["n"], pixel(case), directions(case), receivers(case), precision=case["prec"])
        if case.get("dim") != 3:
            op.autotune()
    _handles[key] = op
    return op


def prepare(case, seed):
    state = {k: v.to(DEV) for k, v in inputs(case, seed).items()}
    state["op"] = handle(case)
    state["case"] = case
    return state


def run(s):
    case, op = s["case"], s["op"]
    k = case["kind"]
    if k == "op":
        return op.apply_A(s["f"], s["x"], adjoint=case["adj"])
    if k in ("forward", "grad", "vec"):
        from paper_1708_01663_amd.cisor import SolveOpts
        opts = SolveOpts(tol=case["tol"], start=1)
    if k == "forward":
        u, y, _, _ = op.forward(s["f"], opts)
        return dict(u=u, y=y)
    if k == "grad":
        g, D, u, v, _, _ = op.grad(s["f"], s["y"], opts)
        return dict(g=g, D=D, u=u, v=v)
    if k == "data":
        w, D = op.project(s["f"], s["u"], s["y"])
        return dict(w=w, D=D, q=op.backproject(w))
    if k == "tv":
        return op.tv_prox(s["z"], TV_LAM, 0.0, 2.0, INNER)
    if k == "vec":
        g, D, _, _, _ = op.grad(s["f"], s["y"], opts)
        return dict(g=g, D=D)
    if k == "predict":
        return op.predict(s["f"], s["ui"], s["ub"])
    L, g = op.loss_grad(s["f"], s["ui"], s["u"], s["ub"])
    return dict(loss=L, g=g)


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Inputs read and outputs written once; operations of the transforms (5 P log2 P per line,
    the zero half of the padding included), products and elementwise steps.  A solve counts its
    operator applications at a nominal eight BiCGSTAB iterations."""
    k, n = case["kind"], case["n"]
    rb = 8 if real_t(case) == torch.float64 else 4
    if k in ("predict", "train"):
        specs, lev = net_layers()
        fl = sum(2 * 9 * ci * co * (n // d) ** 2 for (ci, co, _), d in zip(specs, lev)) * case["B"]
        P = sum(9 * ci * co + co for ci, co, _ in specs)
        io = case["B"] * n * n * (4 + 8 + 8 + 8)
        return dict(bytes=io + 2 * P, flops=fl) if k == "predict" else dict(bytes=io + 6 * P, flops=3 * fl)
    if k == "tv":
        N = n ** case["dim"]
        return dict(bytes=2 * rb * N, flops=INNER * N * (25 if case["dim"] == 2 else 36))
    dim = case.get("dim", 3 if k == "vec" else 2)
    N, T, M = n ** dim, case["T"], case.get("M", 0)
    F = T * (3 if k == "vec" else 1)
    conv = F * 2 * 5 * (2 * n) ** dim * dim * math.log2(2 * n)
    c = 2 * rb
    if k == "op":
        return dict(bytes=2 * c * F * N + rb * N, flops=conv)
    gemm = 8 * M * F * N
    K = N * (3 if k == "vec" else 1)
    if k == "data":
        return dict(bytes=c * (2 * F * N + M * N + 3 * T * M) + rb * N, flops=2 * gemm)
    solve = 16 * conv + 8 * 60 * F * N
    if k == "forward":
        return dict(bytes=c * (2 * F * N + M * K + T * M) + rb * N, flops=solve + gemm)
    return dict(bytes=c * (3 * F * N + M * K + T * M) + 2 * rb * N, flops=2 * solve + 2 * gemm + conv)


# ---------------------------------------------------------------- the same outputs in 64 bits
def hankel(nu, x):
    """Hankel function H_nu (first kind) of order 0 or 1 for x > 0.3, to 1e-14: Hankel's integral
    ((2 / pi x)^(1/2) e^(i (x - nu pi/2 - pi/4)) / Gamma(nu + 1/2)) int_0^inf e^-t t^(nu - 1/2)
    (1 + i t / 2x)^(nu - 1/2) dt by the trapezoidal rule in s = t^(1/2).  (torch's own Bessel
    functions are off by up to 8e-7 from x = 5 on.)"""
    step = 0.085
    acc = torch.zeros_like(x, dtype=torch.complex128)
    for m in range(74):
        s2 = (m * step) ** 2
        q = torch.sqrt(torch.complex(torch.ones_like(x), s2 / (2 * x)))
        wt = (1.0 if m == 0 else 2.0) * step * math.exp(-s2)
        acc += wt / q if nu == 0 else wt * s2 * q
    ph = x - (0.25 + 0.5 * nu) * math.pi
    return torch.polar(torch.sqrt(2 / (math.pi * x)), ph) * acc / (math.sqrt(math.pi) / (1 if nu == 0 else 2))


def kernel2(rho, h):
    """k^2 times the 2D Green's function integrated over the disk of a pixel's area (wavelength 1)."""
    kb = 2 * math.pi
    ka = kb * h / math.sqrt(math.pi)
    h1 = complex(hankel(1, torch.tensor([ka], dtype=torch.float64))[0])
    self_val = torch.tensor(0.5j * math.pi * ka * h1 - 1.0, dtype=torch.complex128, device=rho.device)
    far = (0.5j * math.pi * ka * h1.real) * hankel(0, kb * rho.clamp_min(h))
    return torch.where(rho == 0, self_val, far)


def kernel3(d, h):
    """The same in 3D, over the ball of a voxel's volume."""
    kb = 2 * math.pi
    ka = kb * h * (3 / (4 * math.pi)) ** (1 / 3)
    e = complex(math.cos(ka), math.sin(ka))
    self_val = (1 - 1j * ka) * e - 1
    dd = d.clamp_min(1e-3 * h)
    far = (math.sin(ka) - ka * math.cos(ka)) / kb * torch.polar(1 / dd, kb * dd)
    return torch.where(d == 0, torch.tensor(self_val, dtype=torch.complex128), far)


def spectrum(n, dim, h, dev):
    P = 2 * n
    j = torch.arange(P, dtype=torch.float64)
    d = torch.minimum(j, P - j)
    sq = (h * d) ** 2
    r2 = sq[:, None] + sq[None, :] if dim == 2 else sq[:, None, None] + sq[None, :, None] + sq[None, None, :]
    K = (kernel2 if dim == 2 else kernel3)(r2.sqrt(), h)
    for ax in range(dim):          # offset n never occurs between two cells
        K.select(ax, n).zero_()
    return torch.fft.fftn(K).to(dev)


def convolve(G, x, conj=False):
    """Convolution of fields [T, n, ..., n] by the kernel of spectrum G, some fields at a time."""
    n, dim = x.shape[-1], G.dim()
    ax = tuple(range(-dim, 0))
    out = torch.empty_like(x)
    step = max(1, int(2 ** 26 // G.numel()))
    Gc = G.conj() if conj else G
    crop = (Ellipsis,) + (slice(0, n),) * dim
    for t in range(0, x.shape[0], step):
        out[t:t + step] = torch.fft.ifftn(torch.fft.fftn(x[t:t + step], s=(2 * n,) * dim, dim=ax) * Gc, dim=ax)[crop]
    return out


def solve64(A, b, tol=1e-12, maxit=400):
    """BiCGSTAB on every row of b at once."""
    dot = lambda p, q: (p.conj() * q).sum(1, keepdim=True)  # noqa: E731
    x = torch.zeros_like(b)
    r, rh = b.clone(), b.clone()
    rho = al = om = torch.ones(b.shape[0], 1, dtype=b.dtype, device=b.device)
    v = p = torch.zeros_like(b)
    bn = torch.linalg.vector_norm(b, dim=1, keepdim=True)
    for _ in range(maxit):
        run_ = torch.linalg.vector_norm(r, dim=1, keepdim=True) > tol * bn
        if not bool(run_.any()):
            break
        keep = lambda new, old: torch.where(run_, new, old)  # noqa: E731
        rho1 = dot(rh, r)
        beta = keep(rho1 / rho * al / om, torch.zeros_like(rho))
        p = keep(r + beta * (p - om * v), p)
        rho = keep(rho1, rho)
        v = A(p)
        al = keep(rho / dot(rh, v), al)
        s = r - al * v
        t = A(s)
        om = keep(dot(t, s) / dot(t, t).real.clamp_min(1e-300), om)
        x = keep(x + al * p + om * s, x)
        r = keep(s - om * t, r)
    return x


def grad_div(F, h):
    """(D F)_i = sum_j d_i d_j F_j on [T, 3, n, n, n], zero outside the grid."""
    P = torch.nn.functional.pad(torch.view_as_real(F).movedim(-1, 0), (1,) * 6)
    P = torch.complex(P[0], P[1])
    n = F.shape[-1]

    def at(c, off):
        return P[(slice(None), c) + tuple(slice(1 + o, 1 + o + n) for o in off)]

    out = []
    for i in range(3):
        e = [[int(a == b) for b in range(3)] for a in range(3)]
        acc = at(i, e[i]) - 2 * at(i, (0, 0, 0)) + at(i, [-o for o in e[i]])
        for j in range(3):
            if j != i:
                for a in (1, -1):
                    for b in (1, -1):
                        acc = acc + a * b / 4 * at(j, [a * p + b * q for p, q in zip(e[i], e[j])])
        out.append(acc / h ** 2)
    return torch.stack(out, 1)


def exact(case, seed):
    dev = DEV if torch.cuda.is_available() else "cpu"
    i = {k: v.to(dev).to(torch.complex128 if v.is_complex() else torch.float64)
         for k, v in inputs(case, seed).items()}
    k, n, h = case["kind"], case["n"], pixel(case)
    if k in ("predict", "train"):
        return exact_net(case, i)
    if k == "tv":
        return exact_tv(i["z"].view((n,) * case["dim"]), TV_LAM).reshape(-1)
    if k == "vec":
        return exact_vec(case, i, dev)
    dim = case.get("dim", 2)
    f = i["f"].view((n,) * dim)
    if k != "data":
        G = spectrum(n, dim, h, dev)
        T = case["T"]

        def fwd(x):
            x = x.view((T,) + (n,) * dim)
            return (x - convolve(G, f * x)).reshape(T, -1)

        def adj(x):
            x = x.view((T,) + (n,) * dim)
            return (x - f * convolve(G, x, True)).reshape(T, -1)
    if k == "op":
        return (adj if case["adj"] else fwd)(i["x"])
    ax = (torch.arange(n, dtype=torch.float64) - (n - 1) / 2) * h
    gx = ax.to(dev)
    H = torch.stack([kernel2(torch.hypot(r[0] - gx[:, None], r[1] - gx[None, :]), h).reshape(-1)
                     for r in receivers(case).tolist()])
    f = i["f"]
    if k == "data":
        w = (i["u"] * f) @ H.T - i["y"]
        return dict(w=w, D=0.5 * float(w.abs().square().sum()), q=w @ H.conj())
    f = f.view(n, n)
    d = torch.as_tensor(directions(case))
    ph = 2 * math.pi * (d[:, :1, None] * ax[None, :, None] + d[:, 1:, None] * ax[None, None, :])
    u = solve64(fwd, torch.polar(torch.ones_like(ph), ph).reshape(len(d), -1).to(dev))
    y = (u * f.reshape(-1)) @ H.T
    if k == "forward":
        return dict(u=u, y=y)
    w = y - i["y"]
    q = w @ H.conj()
    v = solve64(adj, q * f.reshape(-1))
    z = q + convolve(G, v.view(-1, n, n), True).reshape(len(d), -1)
    return dict(g=(u.conj() * z).real.sum(0), D=0.5 * float(w.abs().square().sum()), u=u, v=v)


def exact_tv(z, lam):
    """FGP on the dual, the fixed number of iterations."""
    dim = z.dim()

    def grad(x):
        g = torch.zeros((dim,) + x.shape, dtype=x.dtype, device=x.device)
        for a in range(dim):
            m = x.shape[a]
            g[a].narrow(a, 0, m - 1).copy_(x.narrow(a, 1, m - 1) - x.narrow(a, 0, m - 1))
        return g

    def div(p):
        out = torch.zeros_like(p[0])
        for a in range(dim):
            m = p.shape[a + 1]
            out.narrow(a, 0, m - 1).add_(p[a].narrow(a, 0, m - 1))
            out.narrow(a, 1, m - 1).sub_(p[a].narrow(a, 0, m - 1))
        return out

    p = torch.zeros((dim,) + z.shape, dtype=z.dtype, device=z.device)
    r, t = p.clone(), 1.0
    for _ in range(INNER):
        v = r + grad((z + lam * div(r)).clamp(0.0, 2.0)) / (4 * dim * lam)
        new = v / v.square().sum(0).sqrt().clamp_min(1.0)
        t1 = (1 + math.sqrt(1 + 4 * t * t)) / 2
        r, p, t = new + (t - 1) / t1 * (new - p), new, t1
    return (z + lam * div(p)).clamp(0.0, 2.0)


def exact_vec(case, i, dev):
    n, T, h, k0 = case["n"], case["T"], pixel(case), 2 * math.pi
    f = i["f"].view(n, n, n)
    G = spectrum(n, 3, h, dev)
    shape = (T, 3, n, n, n)

    def fwd(x):
        x = x.view(shape)
        Y = convolve(G, (f * x).view(-1, n, n, n)).view(shape)
        return (x - Y - grad_div(Y, h) / k0 ** 2).reshape(T, -1)

    def back(x):
        return convolve(G, (x + grad_div(x, h) / k0 ** 2).view(-1, n, n, n), True).view(shape)

    def adj(x):
        x = x.view(shape)
        return (x - f * back(x)).reshape(T, -1)

    ax = (torch.arange(n, dtype=torch.float64) - (n - 1) / 2) * h
    pos = torch.stack(torch.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    d = torch.as_tensor(directions(case))
    d = d / d.norm(dim=1, keepdim=True)
    pol = torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64) - d[:, 2:] * d
    pol = pol / pol.norm(dim=1, keepdim=True)
    ph = k0 * d @ pos.T
    Ein = (pol[:, :, None] * torch.polar(torch.ones_like(ph), ph)[:, None]).reshape(T, -1).to(dev)
    R = torch.as_tensor(receivers(case))[:, None] - pos[None]
    r = R.norm(dim=2)
    kr = k0 * r
    a = torch.complex(3 / kr ** 2 - 1, -3 / kr)
    b = torch.complex(1 - 1 / kr ** 2, 1 / kr)
    row = a[..., None] * (R / r[..., None]) * (R[..., 2:] / r[..., None])
    row[..., 2] += b
    H = (h ** 3 * k0 ** 2 * torch.polar(1 / (4 * math.pi * r), kr)[..., None] * row).movedim(-1, 1)
    H = H.reshape(case["M"], -1).to(dev)
    f3 = i["f"].repeat(3)
    E = solve64(fwd, Ein)
    w = (E * f3) @ H.T - i["y"]
    q = w @ H.conj()
    V = solve64(adj, q * f3)
    z = q + back(V.view(shape)).reshape(T, -1)
    return dict(g=(E.conj() * z).real.view(T, 3, -1).sum((0, 1)), D=0.5 * float(w.abs().square().sum()))


def net_layers(base=32):
    c1, c2, c3, c4 = base, 2 * base, 4 * base, 8 * base
    specs = [(32, c1, 1), (c1, c1, 1), (c1, c2, 1), (c2, c2, 1), (c2, c3, 1), (c3, c3, 1), (c3, c4, 1), (c4, c4, 1),
             (c3 + c4, c3, 1), (c3, c3, 1), (c2 + c3, c2, 1), (c2, c2, 1), (c1 + c2, c1, 1), (c1, c1, 1), (c1, 32, 0)]
    return specs, [1, 1, 2, 2, 4, 4, 8, 8, 4, 4, 2, 2, 1, 1, 1]


def exact_net(case, i):
    """The network in 64 bits; each 3x3 convolution as nine products."""
    from paper_1708_01663_amd.warmstart import DEFAULT_WEIGHTS
    n, B, dev = case["n"], case["B"], i["f"].device
    par = torch.as_tensor(np.load(DEFAULT_WEIGHTS, allow_pickle=False)["params"]).to(dev).double()
    par.requires_grad_(case["kind"] == "train")
    specs, _ = net_layers()
    layers, off = [], 0
    for ci, co, relu in specs:
        layers.append((par[off:off + 9 * ci * co].view(9, co, ci), par[off + 9 * ci * co:off + (9 * ci + 1) * co], relu))
        off += (9 * ci + 1) * co

    def conv(l, x):                      # x [B, H, W, C]
        w, b, relu = layers[l]
        H, W, C = x.shape[1:]
        p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
        y = b.expand(B * H * W, -1)
        for t in range(9):
            y = y + p[:, t // 3:t // 3 + H, t % 3:t % 3 + W].reshape(-1, C) @ w[t].T
        return (torch.relu(y) if relu else y).view(B, H, W, -1)

    def pool(x):
        return (x[:, ::2, ::2] + x[:, ::2, 1::2] + x[:, 1::2, ::2] + x[:, 1::2, 1::2]) / 4

    def cat(a, b):
        return torch.cat([a, b.repeat_interleave(2, 1).repeat_interleave(2, 2)], 3)

    x = torch.zeros(B, n, n, 32, dtype=torch.float64, device=dev)
    for c, v in enumerate((i["f"], i["ui"].real, i["ui"].imag, i["ub"].real, i["ub"].imag)):
        x[..., c] = v.view(B, n, n)
    with torch.set_grad_enabled(case["kind"] == "train"):
        e1 = conv(1, conv(0, x))
        e2 = conv(3, conv(2, pool(e1)))
        e3 = conv(5, conv(4, pool(e2)))
        bt = conv(7, conv(6, pool(e3)))
        d3 = conv(9, conv(8, cat(e3, bt)))
        d2 = conv(11, conv(10, cat(e2, d3)))
        o = conv(14, conv(13, conv(12, cat(e1, d2)))).view(B, n * n, 32)
        if case["kind"] == "predict":
            return i["ui"] + torch.complex(o[..., 0], o[..., 1])
        t = i["u"] - i["ui"]
        e = (o[..., 0] - t.real).square() + (o[..., 1] - t.imag).square()
        loss = (e.sum(1) / t.abs().square().sum(1)).mean()
        loss.backward()
    return dict(loss=float(loss.detach()), g=par.grad)
