"""Workloads on which the library's speed is judged.

Each case is one pass through public entry points of paper_1007_3432_amd.hub
on one lattice: a conjugate-gradient solve, a preconditioned solve, a
molecular-dynamics trajectory, a product with Q = M^T M, the single operators
around a solve, or a batch of served solves.  Fields of a case:

  kind      "cg" | "pcg" | "md" | "mtm" | "ops" | "serve"
  d, nx, nt lattice (t = 1, dtau = 0.05, U = -2, mu = 0 everywhere)
  prec      "f64" | "f32" | "f16": vectors and links in FP64, in FP32, or FP32
            vectors with FP16 links (for solves: the bulk precision)
  n, eps    pcg: half-degree and interval; md: steps and step size;
            serve: n solves over the serving lattices, d/nx/nt being unused

The field sigma is uniform on [-pi, pi) and the source of a solve is
phi = M^T eta with eta standard normal, as everywhere in this repository.
Solves go to a relative residual of 1e-12: molecular dynamics has to retrace
its path, and the error of x is the residual's times a factor that grows with
the extent in time (500 at 128 slices), so that x is then good to nine digits.
"""
import math
import time

import numpy as np
import torch

from paper_1007_3432_amd import hub, inputs

DEV = "cuda"
T_HOP, DTAU, U = 1.0, 0.05, -2.0
KAPPA = DTAU * T_HOP
B = math.sqrt(2.0 * (math.exp(-DTAU * U) - 1.0))
PREC = {"f64": (hub.F64, hub.F64), "f32": (hub.F32, hub.F32), "f16": (hub.F32, hub.F16)}
MAX_ITER = 1000000
TOL = 1e-12


def listed():
    return [
        # The smallest solve in earnest: the benchmark's HMC chain and the smoke test run on it.
        dict(name="cg_f64_d1_32x64", kind="cg", d=1, nx=32, nt=64, prec="f64"),
        # A long chain in FP64: half a million sites.
        dict(name="cg_f64_d1_4096x128", kind="cg", d=1, nx=4096, nt=128, prec="f64"),
        # The middle of the matrix-vector experiment's d = 3 lattices, the usual production size.
        dict(name="cg_f64_d3_16x128", kind="cg", d=3, nx=16, nt=128, prec="f64"),
        # A two-dimensional lattice with an odd extent: no size in it is a power of two.
        dict(name="cg_f64_d2_33x60", kind="cg", d=2, nx=33, nt=60, prec="f64"),
        # A large lattice in mixed precision with compact links, as the benchmark solves its largest.
        dict(name="cg_f16_d3_32x128", kind="cg", d=3, nx=32, nt=128, prec="f16"),
        # The paper's solver: CG preconditioned by a Chebyshev polynomial, at the benchmark's best degree.
        dict(name="pcg_f64_d3_16x128", kind="pcg", d=3, nx=16, nt=128, prec="f64", n=16, eps=4e-4),
        # A leapfrog trajectory, a solve for each force: what an HMC program spends its time on.
        dict(name="md_f64_d3_8x80", kind="md", d=3, nx=8, nt=80, prec="f64", n=4, eps=0.02),
        # The matrix-vector product by itself: the benchmark's headline, streamed.
        dict(name="mtm_f64_d1_2048x512", kind="mtm", d=1, nx=2048, nt=512, prec="f64"),
        # The same on the largest lattice of the benchmark.
        dict(name="mtm_f64_d3_32x256", kind="mtm", d=3, nx=32, nt=256, prec="f64"),
        # Compact precision on an extent that no tile divides.
        dict(name="mtm_f16_d3_20x96", kind="mtm", d=3, nx=20, nt=96, prec="f16"),
        # The short calls around a solve, where launches count: links, heatbath, force.
        dict(name="ops_f64_d1_256x128", kind="ops", d=1, nx=256, nt=128, prec="f64"),
        # Solves of several HMC chains served together, fields and sources in host memory.
        dict(name="serve_f32_8", kind="serve", d=0, nx=0, nt=0, prec="f32", n=8, eps=0.0),
    ]


def _draw_lattice(rng, lo, hi, nt_hi):
    """d, nx, nt with lo <= volume <= hi, volume and slices spread over their logarithms; half of the
    extents are the round ones that configurations use, the others any."""
    while True:
        d = rng.choice([1, 2, 3])
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        nt = int(round(math.exp(rng.uniform(math.log(4), math.log(nt_hi)))))
        nx = max(2, int(round((v / nt) ** (1.0 / d))))
        if rng.random() < 0.5:
            nx = 2 ** max(1, round(math.log2(nx)))
        if lo <= nx ** d * nt <= hi:
            return dict(d=d, nx=nx, nt=nt)


def draw(rng):
    kind = rng.choice(["cg", "cg", "mtm", "mtm", "pcg", "md", "ops", "serve"])
    if kind == "cg":
        return dict(kind=kind, prec=rng.choice(["f64", "f64", "f32", "f16"]), **_draw_lattice(rng, 500, 1 << 20, 128))
    if kind == "pcg":
        return dict(kind=kind, prec="f64", n=rng.choice([4, 8, 16, 32]), eps=rng.choice([1e-4, 4e-4, 1.6e-3]),
                    **_draw_lattice(rng, 4000, 1 << 20, 128))
    if kind == "md":
        return dict(kind=kind, prec=rng.choice(["f64", "f64", "f32"]), n=rng.randint(2, 6), eps=rng.choice([0.01, 0.02]),
                    **_draw_lattice(rng, 500, 100000, 80))
    if kind == "mtm":
        return dict(kind=kind, prec=rng.choice(["f64", "f64", "f32", "f16"]), **_draw_lattice(rng, 2000, 1 << 23, 512))
    if kind == "ops":
        return dict(kind=kind, prec="f64", **_draw_lattice(rng, 2000, 1 << 23, 512))
    return dict(kind=kind, d=0, nx=0, nt=0, prec=rng.choice(["f32", "f16"]), n=rng.randint(2, 12), eps=0.0)


# --- the operator in plain torch (FP64): inputs of the solves and the exact results

def _shape(d, nx, nt):
    return (nt,) + (nx,) * d


def _links(sigma):
    """A_s = -(1 + b sin sigma_{s-1}), + on slice 0, from sigma of shape (nt, nx, ...)."""
    a = -(1.0 + B * torch.sin(torch.roll(sigma, 1, 0)))
    a[0] = -a[0]
    return a


def _hop(v):
    h = torch.zeros_like(v)
    for k in range(1, v.dim()):
        h += torch.roll(v, 1, k)
        h += torch.roll(v, -1, k)
    return h


def _M(a, v):
    return v - KAPPA * _hop(v) + a * torch.roll(v, 1, 0)


def _Mt(a, v):
    return v - KAPPA * _hop(v) + torch.roll(a * v, -1, 0)


def _Q(a, v):
    return _Mt(a, _M(a, v))


def _cg(a, f, x, tol, most):
    """Plain CG from x until |f - Q x| has fallen by about `tol`."""
    r = f - _Q(a, x)
    p, rho = r.clone(), (r * r).sum()
    stop = float(rho) * tol * tol
    for it in range(1, most + 1):
        q = _Q(a, p)
        alpha = rho / (p * q).sum()
        x = x + alpha * p
        r = r - alpha * q
        new = (r * r).sum()
        p = r + (new / rho) * p
        rho = new
        if it % 50 == 0 and not float(rho) > stop:
            break
    return x


def _solve(a, f):
    """Q^{-1} f, refined once so that rounding in the first solve does not show."""
    x = _cg(a, f, torch.zeros_like(f), 1e-13, MAX_ITER)
    return _cg(a, f, x, 1e-3, MAX_ITER)


def _force(sigma, x):
    a = _links(sigma)
    y = torch.roll(_M(a, x), -1, 0)
    sign = -torch.ones_like(sigma)
    sign[-1] = 1.0
    return -2.0 * y * sign * B * torch.cos(sigma) * x


def _fields(d, nx, nt, seed, count):
    """sigma and `count` standard normal vectors, made on the GPU from the seed."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    s = _shape(d, nx, nt)
    sigma = (torch.rand(s, dtype=torch.float64, device=DEV, generator=g) * 2.0 - 1.0) * math.pi
    return [sigma] + [torch.randn(s, dtype=torch.float64, device=DEV, generator=g) for _ in range(count)]


def _serve_problem(k, seed):
    """Chain k of a served batch: lattice by turns, sigma and eta."""
    shape = inputs.SERVE_SHAPES[k % len(inputs.SERVE_SHAPES)]
    return (shape,) + tuple(_fields(*shape, seed * 64 + k, 1))


# --- what is timed

def prepare(case, seed):
    kind, prec = case["kind"], case["prec"]
    vec, link = PREC[prec]
    if kind == "serve":
        chains = []
        for k in range(case["n"]):
            shape, sigma, eta = _serve_problem(k, seed)
            phi = _Mt(_links(sigma), eta)
            chains.append((hub.lattice(*shape), sigma.cpu().numpy().reshape(-1), phi.cpu().numpy().reshape(-1)))
        opts = hub.cg_opts(hub.F32, link, tol=TOL, max_iter=MAX_ITER)
        return dict(case=case, chains=chains, server=hub.Server(32 << 30, 64, opts))
    d, nx, nt = case["d"], case["nx"], case["nt"]
    s = dict(case=case, lat=hub.lattice(d, nx, nt, T_HOP, DTAU, U))
    if kind in ("cg", "pcg"):
        sigma, eta = _fields(d, nx, nt, seed, 1)
        phi = _Mt(_links(sigma), eta)
        s.update(sigma=sigma.view(-1), phi=phi.view(-1), x=torch.empty_like(phi).view(-1),
                 opts=hub.cg_opts(vec, link, tol=TOL, max_iter=MAX_ITER))
        if kind == "pcg":
            s["cheb"] = hub.cheb_opts(case["n"], case["eps"])
    elif kind == "md":
        sigma, eta, pi = _fields(d, nx, nt, seed, 2)
        phi = _Mt(_links(sigma), eta / math.sqrt(2.0))
        s.update(sigma=sigma.view(-1), pi=pi.view(-1), phi=phi.view(-1),
                 opts=hub.md_opts(case["n"], case["eps"], hub.cg_opts(vec, link, tol=TOL, max_iter=MAX_ITER)))
    elif kind == "mtm":
        sigma, x = _fields(d, nx, nt, seed, 1)
        x = x.to(hub._torch_dtype(vec)).view(-1)
        links = torch.empty(sigma.numel(), dtype=hub._torch_dtype(link), device=DEV)
        hub.hub_links_from_sigma(s["lat"], sigma.view(-1), links, link)
        s.update(links=links, x=x, z=torch.empty_like(x))
    else:
        sigma, eta, x = _fields(d, nx, nt, seed, 2)
        s.update(sigma=sigma.view(-1), eta=eta.view(-1), x=x.view(-1))
        s.update({k: torch.empty_like(s["sigma"]) for k in ("links", "phi", "force")})
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "serve":
        srv = s["server"]
        tickets = [srv.submit(k, lat, sigma, phi) for k, (lat, sigma, phi) in enumerate(s["chains"])]
        out = [None] * len(tickets)
        while True:
            for k, t in enumerate(tickets):
                if out[k] is None:
                    r = srv.poll(t, s["chains"][k][0].volume)
                    if r is not None:
                        out[k] = r[0]
            if all(o is not None for o in out):
                return out
            time.sleep(0.0005)
    lat = s["lat"]
    if kind == "cg":
        hub.hub_cg_solve(lat, s["sigma"], s["phi"], s["x"], s["opts"])
        return s["x"]
    if kind == "pcg":
        hub.hub_pcg_solve(lat, s["sigma"], s["phi"], s["x"], s["opts"], s["cheb"])
        return s["x"]
    if kind == "md":
        sigma, pi = s["sigma"].clone(), s["pi"].clone()
        st = hub.hub_md_trajectory(lat, sigma, pi, s["phi"], s["opts"])
        return dict(sigma=sigma, pi=pi, h_start=st["h_start"], h_end=st["h_end"])
    if kind == "mtm":
        vec, link = PREC[case["prec"]]
        hub.hub_apply_MtM(lat, s["links"], link, vec, s["x"], s["z"])
        return s["z"]
    hub.hub_links_from_sigma(lat, s["sigma"], s["links"], hub.F64)
    hub.hub_apply_M(lat, s["links"], hub.F64, hub.F64, s["eta"], s["phi"], 1)
    hub.hub_hmc_force(lat, s["sigma"], s["x"], s["force"])
    return dict(links=s["links"], phi=s["phi"], force=s["force"])


def _iters(nt):
    """Applications of Q that a solve needs, roughly: they grow with the extent in time."""
    return 50 * nt


def work(case):
    kind, d = case["kind"], case["d"]
    if kind == "serve":
        shapes = [inputs.SERVE_SHAPES[k % len(inputs.SERVE_SHAPES)] for k in range(case["n"])]
        return dict(bytes=sum(24 * inputs.volume(*s) for s in shapes),
                    flops=sum((8 * s[0] + 20) * inputs.volume(*s) * _iters(s[2]) for s in shapes))
    V = case["nx"] ** d * case["nt"]
    q = 8 * d + 10          # operations of Q at a site: two stencils of 2d + 2 products and sums
    if kind == "mtm":
        return dict(bytes={"f64": 24, "f32": 12, "f16": 10}[case["prec"]] * V, flops=q * V)
    if kind == "ops":
        return dict(bytes=64 * V, flops=(8 * d + 40) * V)
    solve = (q + 10) * V * _iters(case["nt"])
    if kind == "md":
        return dict(bytes=40 * V, flops=(case["n"] + 1) * solve)
    return dict(bytes=24 * V, flops=solve)


def exact(case, seed):
    kind = case["kind"]
    if kind == "serve":
        if case["n"] > 8:
            return None
        out = []
        for k in range(case["n"]):
            _, sigma, eta = _serve_problem(k, seed)
            a = _links(sigma)
            out.append(_solve(a, _Mt(a, eta)).view(-1))
        return out
    d, nx, nt = case["d"], case["nx"], case["nt"]
    if kind in ("cg", "pcg"):
        if nx ** d * nt > 3 << 20:
            return None     # plain torch takes too long
        sigma, eta = _fields(d, nx, nt, seed, 1)
        a = _links(sigma)
        return _solve(a, _Mt(a, eta)).view(-1)
    if kind == "md":
        sigma, eta, pi = _fields(d, nx, nt, seed, 2)
        phi = _Mt(_links(sigma), eta / math.sqrt(2.0))
        eps = case["eps"]
        h = []
        for k in range(case["n"] + 1):
            x = _solve(_links(sigma), phi)
            f = _force(sigma, x)
            if k == 0:
                h.append(float(0.5 * (pi * pi).sum() + (phi * x).sum()))
            pi = pi - (0.5 if k in (0, case["n"]) else 1.0) * eps * f
            if k < case["n"]:
                sigma = sigma + eps * pi
        h.append(float(0.5 * (pi * pi).sum() + (phi * x).sum()))
        return dict(sigma=sigma.view(-1), pi=pi.view(-1), h_start=h[0], h_end=h[1])
    if kind == "mtm":
        vec, _ = PREC[case["prec"]]
        sigma, x = _fields(d, nx, nt, seed, 1)
        if case["prec"] == "f16":
            sn = torch.sin(torch.roll(sigma, 1, 0)).to(torch.float16).double()
            a = -(1.0 + B * sn)
            a[0] = -a[0]
        else:
            a = _links(sigma)
        return _Q(a, x.to(hub._torch_dtype(vec)).double()).view(-1)
    sigma, eta, x = _fields(d, nx, nt, seed, 2)
    a = _links(sigma)
    return dict(links=a.view(-1), phi=_Mt(a, eta).view(-1), force=_force(sigma, x).view(-1))
