"""Timed workloads of the planar photoacoustic operator.

Each case is one piece of work that a program using the package does through
its public entry points (``Operator``, ``autograd``, ``serve.Server``):

    listed()             the standing cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs, library and handle a program holds beforehand
    run(state)           one pass; returns every output of the pass
    work(case)           bytes and operations the pass cannot do without
    exact(case, seed)    the same outputs in 64-bit arithmetic, by plain torch

Kinds of work:

    pair   A x and A^T d, the two applies every gradient of a reconstruction
           needs (B objects at a time)
    grad   1/2 ||A x - d||^2 and its gradient through torch.autograd
    fista  ``recon_fista``: a whole reconstruction from measured data
    serve  B requests of one class through the continuous-batching server,
           from submission to the last result
    cold   a new geometry: library build, step size by power iteration, then
           a reconstruction

Objects are Gaussian absorbers and data are their closed-form free-space
pressure at the sensor plane plus 1 % noise, so that values and their
distribution over depth and time are those of photoacoustic data.  The
physics is that of the synthetic workloads used throughout the repository
(dx = dy = dz = 100 um, c = 1500 m/s, dt = 0.3 dx / c).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2603_28150_amd import autograd
from paper_2603_28150_amd.op import Geometry, Operator
from paper_2603_28150_amd.serve import HipBackend, Request, Server

CFL = 0.3
FAST_SIZES = (16, 32, 48, 64, 72, 96, 108, 128, 144, 192, 216, 256, 288, 384, 432, 512, 576, 768, 864, 1024)
NOISE = 0.01
POWER_ITERATIONS = 30


def _case(kind, nx, ny, nz, nt, dtype="f32", batch=1, boundary="periodic", step=1, niter=0, name=None):
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, nt=nt, dtype=dtype, batch=batch, boundary=boundary,
             step=step, niter=niter)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a first try or a unit-sized problem, bound by launches
        _case("pair", 32, 32, 16, 64, name="pair_32_f32"),
        # the smallest served class, one object at a time
        _case("pair", 64, 64, 64, 256, name="pair_64_f32"),
        # one step of a torch-side optimiser (learned or TV-regularised reconstruction)
        _case("grad", 128, 128, 64, 256, name="grad_128_f32"),
        # the benchmark's step: the full-size operator pair of one object
        _case("pair", 256, 256, 128, 512, name="pair_256_f32"),
        # the same with the 16-bit library (half the memory per geometry)
        _case("pair", 256, 256, 128, 512, dtype="bf16", name="pair_256_bf16"),
        # a data set of many objects on one geometry: the largest call
        _case("pair", 256, 256, 128, 512, batch=16, name="pair_256_f32_b16"),
        # the same for a mid-size geometry on the 16-bit library
        _case("pair", 128, 128, 96, 384, dtype="bf16", batch=8, name="pair_128_bf16_b8"),
        # the wire-phantom grid with the zero-padded (linear) convolution: odd
        # depth count, rows that are not whole 16-byte units
        _case("pair", 202, 202, 37, 256, boundary="linear", name="pair_202_linear"),
        # the same grid taken as periodic: an axis length that is no fast transform size
        _case("pair", 202, 202, 37, 256, name="pair_202_periodic"),
        # a full-size reconstruction
        _case("fista", 256, 256, 128, 512, niter=50, name="fista_256_f32"),
        # served reconstructions: four requests of one class
        _case("serve", 128, 128, 96, 384, dtype="bf16", batch=4, niter=20, name="serve_128_bf16"),
        # first reconstruction on a new geometry
        _case("cold", 128, 128, 96, 384, niter=20, name="cold_128_f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    """Rough seconds of a pass, to keep drawn cases below the largest listed
    one (a library build runs in 64-bit arithmetic: several times the cost of
    the float32 passes)."""
    w = work(case)
    return (w["bytes"] / 5e12 + w["flops"] / 50e12) * (6.0 if case["kind"] == "cold" else 1.0)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= most:
            return c


def _draw(rng):
    kind = rng.choice(["pair", "pair", "pair", "pair", "grad", "fista", "serve", "cold"])
    fast = [n for n in FAST_SIZES if n <= 256]
    boundary = "linear" if kind in ("pair", "grad", "fista") and rng.random() < 0.25 else "periodic"
    if boundary == "linear":
        nx, ny = _log_int(rng, 16, 216), _log_int(rng, 16, 216)
        if rng.random() < 0.5:
            ny = nx
    elif kind == "pair" and rng.random() < 0.2:
        nx = 2 * _log_int(rng, 8, 128)  # any even length
        ny = nx if rng.random() < 0.5 else rng.choice(fast)
    else:
        nx = rng.choice(fast)
        ny = nx if rng.random() < 0.7 else rng.choice(fast)
    nz, nt = _log_int(rng, 8, 128), _log_int(rng, 48, 512)
    batch = 1
    if kind == "pair" and rng.random() < 0.4:
        batch = _log_int(rng, 2, 16)
    if kind == "serve":
        batch = rng.randint(1, 8)
    dtype = rng.choice(["f32", "f32", "bf16", "f16"])
    step = 1
    if kind in ("pair", "fista") and boundary == "periodic" and nx % 8 == 0 and ny % 2 == 0 \
            and nx in FAST_SIZES and ny in FAST_SIZES and rng.random() < 0.15:
        step = 2  # a scan grid at every second point
    niter = rng.randint(5, 20) if kind in ("fista", "serve", "cold") else 0
    return _case(kind, nx, ny, nz, nt, dtype, batch, boundary, step, niter)


# ------------------------------------------------------------------ inputs
def _absorbers(case, seed, b):
    """Centres (z, y, x), widths and amplitudes of object b, in voxels."""
    r = np.random.default_rng([seed, b, 77])
    n = 8
    depth = max(4.0, 0.9 * case["nz"])
    return np.stack([r.uniform(2.0, depth, n), r.uniform(0, case["ny"], n), r.uniform(0, case["nx"], n),
                     r.uniform(1.0, 3.0, n), r.uniform(0.2, 1.0, n)], axis=1).tolist()


def _axes(case, n):
    dev = torch.device("cuda", 0)
    return (torch.arange(n, device=dev, dtype=torch.float32)[:, None, None],
            torch.arange(case["ny"], device=dev, dtype=torch.float32)[None, :, None],
            torch.arange(case["nx"], device=dev, dtype=torch.float32)[None, None, :])


def _objects(case, seed):
    z, y, x = _axes(case, case["nz"])
    out = torch.zeros((case["batch"], case["nz"], case["ny"], case["nx"]), device=z.device)
    for b in range(case["batch"]):
        for cz, cy, cx, s, a in _absorbers(case, seed, b):
            e = (torch.exp((y - cy) ** 2 * (-0.5 / s ** 2)) * torch.exp((x - cx) ** 2 * (-0.5 / s ** 2)))
            out[b] += a * torch.exp((z - cz) ** 2 * (-0.5 / s ** 2)) * e
    return out


def _data(case, seed):
    """Closed-form pressure of the absorbers at the sensor plane, with noise."""
    n, y, x = _axes(case, case["nt"])
    ct = CFL * n
    step = case["step"]
    ys, xs = y[:, ::step], x[:, :, ::step]
    out = torch.zeros((case["batch"], case["nt"], ys.shape[1], xs.shape[2]), device=n.device)
    g = torch.Generator(device=n.device)
    for b in range(case["batch"]):
        for cz, cy, cx, s, a in _absorbers(case, seed, b):
            R = torch.sqrt((ys - cy) ** 2 + (xs - cx) ** 2 + cz * cz)
            for u in (R - ct, R + ct):
                out[b] += u * torch.exp(u * u * (-0.5 / s ** 2)) * (0.5 * a / R)
        g.manual_seed(seed * 1009 + b)
        rms = torch.sqrt(torch.mean(out[b] * out[b]))
        out[b] += torch.randn(out[b].shape, generator=g, device=n.device) * (NOISE * rms)
    return out


def _start_vector(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 5)
    return torch.randn((case["nz"], case["ny"], case["nx"]), generator=g, device="cuda")


def _tau(case):
    # a step below 1/||A||^2 for this physics (||A||^2 grows like sqrt(nt))
    return 1.0 / (1.0 + math.sqrt(case["nt"]))


def _geometry(case):
    return Geometry.paper_like(case["nx"], case["ny"], case["nz"], case["nt"], cfl=CFL,
                               boundary=case["boundary"], sx=case["step"], sy=case["step"])


def _one(case, t):
    return t[0] if case["batch"] == 1 else t


def prepare(case, seed):
    s = dict(case=case, geom=_geometry(case))
    kind = case["kind"]
    if kind == "cold":
        s["d"], s["v0"] = _one(case, _data(case, seed)), _start_vector(case, seed)
        return s
    if kind == "serve":
        s["d"] = _data(case, seed)
        s["server"] = Server(HipBackend(), hbm_budget=64 << 30, max_batch=16)
        # a warm class: library built, pool grown by an earlier group of requests
        _serve(s, 1)
        return s
    s["op"] = Operator(s["geom"], case["dtype"])
    s["d"] = _one(case, _data(case, seed))
    if kind in ("pair", "grad"):
        s["x"] = _one(case, _objects(case, seed + 1))
    return s


# -------------------------------------------------------------------- run
def _serve(s, niter):
    srv, case = s["server"], s["case"]
    reqs = [srv.submit(Request(geom=s["geom"], d=s["d"][b], niter=niter, h_dtype=case["dtype"], tau=_tau(case)))
            for b in range(case["batch"])]
    srv.run_until_idle()
    srv.finished.clear()
    return [r.x for r in reqs]


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "pair":
        return s["op"].apply_A(s["x"]), s["op"].apply_AT(s["d"])
    if kind == "grad":
        x = s["x"].detach().requires_grad_(True)
        r = autograd.forward(s["op"], x) - s["d"]
        loss = 0.5 * (r * r).sum()
        loss.backward()
        return loss.detach(), x.grad
    if kind == "fista":
        return s["op"].recon_fista(s["d"], case["niter"], _tau(case))
    if kind == "serve":
        return _serve(s, case["niter"])
    op = Operator(s["geom"], case["dtype"])
    L, _ = op.power_norm(s["v0"], POWER_ITERATIONS)
    return L, op.recon_fista(s["d"], case["niter"], 1.0 / L)


# ------------------------------------------------------------------- work
def _periods(case):
    if case["boundary"] == "periodic":
        return case["nx"], case["ny"]
    return tuple(min(p for p in FAST_SIZES if p >= max(16, 2 * n)) for n in (case["nx"], case["ny"]))


def _classes(fx, fy):
    """Frequencies with equal transverse wavenumber share one library block:
    (class of every half-spectrum frequency [fy * nh], one (m, p) per class)."""
    m = np.arange(fx // 2 + 1)[None, :]
    p = np.arange(fy)[:, None]
    p = np.minimum(p, fy - p)
    key = m * m + p * p if fx == fy else m * (fy + 1) + p
    _, first, inv = np.unique(key.ravel(), return_index=True, return_inverse=True)
    m, p = np.broadcast_to(m, key.shape).ravel(), np.broadcast_to(p, key.shape).ravel()
    return inv.ravel(), m[first], p[first]


def work(case):
    nx, ny, nz, nt, B, step = (case[k] for k in ("nx", "ny", "nz", "nt", "batch", "step"))
    fx, fy = _periods(case)
    nk = fy * (fx // 2 + 1)
    nclass = len(_classes(fx, fy)[1])
    esz = 4 if case["dtype"] == "f32" else 2
    lib = nclass * nz * nt * esz
    vox, dat = 4 * B * nx * ny * nz, 4 * B * (nx // step) * (ny // step) * nt
    fft = 2.5 * fx * fy * math.log2(fx * fy) * B
    apply_flops = 4.0 * nk * nz * nt * B + fft * (nz + nt)
    if case["kind"] in ("pair", "grad"):
        return {"bytes": 2 * (lib + vox + dat), "flops": 2 * apply_flops}
    # reconstructions: A^T d once, then per iteration the nz x nz normal
    # blocks (symmetric) and the object arrays z, x read and written; where
    # cropping or sampling couples the frequencies, the two applies
    it = case["niter"]
    if case["boundary"] == "linear" or step > 1:
        per, fl = 2 * lib + 4 * vox, 2 * apply_flops
    else:
        per = nclass * nz * (nz + 1) // 2 * 4 + 4 * vox
        fl = 4.0 * nk * nz * nz * B + 2 * fft * nz
    out = {"bytes": lib + vox + dat + it * per, "flops": apply_flops + it * fl}
    if case["kind"] == "cold":
        # the library written (both storage orders are the build's own choice:
        # once), its cosines (20 operations each) and depth sums, then the
        # power iteration
        nq = _z_period(case)
        build = nclass * nt * (nq // 2 + 1) * (20.0 + 2.0 * nz) + 2.0 * nclass * nz * nz * nt
        out["bytes"] += lib + POWER_ITERATIONS * (nclass * nz * (nz + 1) // 2 * 4 + 2 * vox)
        out["flops"] += build + POWER_ITERATIONS * fl
    return out


# ------------------------------------------------------------------ exact
def _z_period(case):
    need = case["nz"] + math.ceil(CFL * (case["nt"] - 1) - 1e-9) + 1
    return 1 << max(0, math.ceil(math.log2(need)))


class _Exact:
    """The operator in 64 bits: the sensor-plane response of every depth as a
    sum over the axial wavenumbers, one block per class of frequencies."""

    def __init__(self, case):
        self.case = case
        self.fx, self.fy = _periods(case)
        self.nh = self.fx // 2 + 1
        inv, m, p = _classes(self.fx, self.fy)
        self.cls = torch.from_numpy(inv).cuda()
        nz, nt, nq = case["nz"], case["nt"], _z_period(case)
        f64 = dict(dtype=torch.float64, device="cuda")
        kx = torch.from_numpy(2 * math.pi * m / self.fx).cuda()
        ky = torch.from_numpy(2 * math.pi * p / self.fy).cuda()
        q = torch.arange(nq // 2 + 1, **f64)
        kz = 2 * math.pi * q / nq
        w = torch.full_like(q, 2.0 / nq)
        w[0] = 1.0 / nq
        if nq % 2 == 0:
            w[-1] = 1.0 / nq
        E = w[:, None] * torch.cos(2 * math.pi * torch.outer(q, torch.arange(nz, **f64)).remainder(nq) / nq)
        n = torch.arange(nt, **f64)
        self.H = torch.empty((len(m), nz, nt), **f64)
        chunk = max(1, (1 << 27) // (nt * len(q)))
        for c in range(0, len(m), chunk):
            th = CFL * torch.sqrt(kx[c:c + chunk, None] ** 2 + ky[c:c + chunk, None] ** 2 + kz[None, :] ** 2)
            ph = torch.cos(n[None, :, None] * th[:, None, :])
            self.H[c:c + chunk] = torch.matmul(ph, E).transpose(1, 2)
        if case["dtype"] != "f32":
            e, kind = (0, torch.bfloat16) if case["dtype"] == "bf16" else (15, torch.float16)
            amax = self.H.abs().amax(dim=(0, 2))
            scale = torch.exp2(e - torch.ceil(torch.log2(amax)))[:, None]
            for c in range(0, len(m), chunk):
                h = self.H[c:c + chunk]
                h.copy_((h * scale).float().to(kind).double() / scale)
        self.G = None

    def _spectrum(self, f):
        F = torch.fft.rfft2(f.double(), s=(self.fy, self.fx))
        return torch.view_as_real(F.reshape(F.shape[0], -1).t().contiguous())  # [nk, n, 2]

    def _slices(self, S):
        F = torch.view_as_complex(S).t().reshape(-1, self.fy, self.nh)
        return torch.fft.irfft2(F, s=(self.fy, self.fx))[:, :self.case["ny"], :self.case["nx"]]

    def _product(self, blocks, S, transpose):
        rows = blocks.shape[2] if transpose else blocks.shape[1]
        out = torch.empty((S.shape[0], rows, 2), dtype=torch.float64, device="cuda")
        chunk = max(1, (1 << 27) // (blocks.shape[1] * blocks.shape[2]))
        for c in range(0, S.shape[0], chunk):
            h = blocks[self.cls[c:c + chunk]]
            out[c:c + chunk] = torch.bmm(h.transpose(1, 2).contiguous() if transpose else h, S[c:c + chunk])
        return out

    def A(self, x):
        step = self.case["step"]
        return self._slices(self._product(self.H, self._spectrum(x), True))[:, ::step, ::step]

    def AT(self, d):
        step = self.case["step"]
        full = torch.zeros((d.shape[0], self.case["ny"], self.case["nx"]), dtype=torch.float64, device="cuda")
        full[:, ::step, ::step] = d
        return self._slices(self._product(self.H, self._spectrum(full), False))

    def normal(self, x):
        if self.case["boundary"] == "linear" or self.case["step"] > 1:
            return self.AT(self.A(x))
        if self.G is None:
            self.G = torch.bmm(self.H, self.H.transpose(1, 2).contiguous())
        return self._slices(self._product(self.G, self._spectrum(x), False))

    def fista(self, d, niter, tau):
        b = self.AT(d)
        x = torch.zeros_like(b)
        z, t = x, 1.0
        for _ in range(niter):
            t_next = (1.0 + math.sqrt(1.0 + 4.0 * t * t)) / 2.0
            new = torch.clamp(z - tau * (self.normal(z) - b), min=0.0)
            z = new + ((t - 1.0) / t_next) * (new - x)
            x, t = new, t_next
        return x

    def norm(self, v, niter):
        v = v.double() / torch.linalg.vector_norm(v.double())
        for _ in range(niter):
            w = self.normal(v)
            L = float((v * w).sum())
            v = w / torch.linalg.vector_norm(w)
        return L


def exact(case, seed):
    op = _Exact(case)
    kind = case["kind"]
    d = _data(case, seed)
    if kind in ("pair", "grad"):
        x = _objects(case, seed + 1)
        if kind == "grad":
            r = op.A(x[0]) - d[0].double()
            return 0.5 * (r * r).sum(), op.AT(r)
        return _one(case, torch.stack([op.A(v) for v in x])), _one(case, torch.stack([op.AT(v) for v in d]))
    if kind == "fista":
        return op.fista(d[0], case["niter"], _tau(case))
    if kind == "serve":
        return [op.fista(v, case["niter"], _tau(case)) for v in d]
    L = op.norm(_start_vector(case, seed), POWER_ITERATIONS)
    return L, op.fista(d[0], case["niter"], 1.0 / L)
