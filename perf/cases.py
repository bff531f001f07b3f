"""Workloads whose speed matters to users of the 3PCF library, each one pass through the public entry points.

A pass starts from what a program holds on the GPU (a catalogue, a plan, and for gradients the cotangent of
the multipoles) and ends with the multipoles and, where asked for, the gradients.  Catalogues are log-normal
mocks (cells drawn with weight exp(G - 1/2), P(k) ~ k^-1.5 exp(-(kR)^2), unit variance on the grid) drawn on the GPU;
"cells" keeps them in grid order, as a mock generator or a sorted snapshot writes them, "random" shuffles them,
as an N-body particle file comes.

The multipoles leave the library as float64 sums; a float32 plan's fields carry float32 accuracy, so its
outputs are handed on in float32, the precision of the plan.
"""
import math

import numpy as np
import torch

import paper_2507_15209_amd as mp3
from paper_2507_15209_amd import autotune


def _case(name, form, call, n, box, lmax, nbins, r_lo, r_hi, particles, precision="f32", smooth=8.0, weights=False,
          order="cells", batch=1, basis="b3", binning="shell", top_hat=0.0, phi_hat=False):
    return {"name": name, "form": form, "call": call, "n": n, "box": box, "lmax": lmax, "nbins": nbins, "r_lo": r_lo,
            "r_hi": r_hi, "particles": particles, "precision": precision, "smooth": smooth, "weights": weights,
            "order": order, "batch": batch, "basis": basis, "binning": binning, "top_hat": top_hat,
            "phi_hat": phi_hat}


def listed():
    return [
        # The smallest survey box in double precision: a gradient evaluated many times in a fit, so launches count.
        _case("nodal_32_f64", "nodal", "sweep", 32, 250.0, 4, 6, 10.0, 60.0, 2000, "f64", 4.0),
        # The same box by the exact grid summation with the connection coefficients.
        _case("gamma_32_f64", "gamma", "sweep", 32, 250.0, 4, 6, 10.0, 60.0, 2000, "f64", 4.0),
        # A catalogue's multipoles with thin shells and a top-hat on every vertex, differentiated by autograd
        # (forward and backward as two calls) in double precision.
        _case("nodal_128_f64_autograd", "nodal", "autograd", 128, 1000.0, 6, 13, 20.0, 150.0, 900_001, "f64",
              weights=True, order="random", binning="thin", top_hat=8.0),
        # The throughput workload: 256^3, L = 10, 20 bins, 8e6 particles, value and gradient.
        _case("nodal_256_f32", "nodal", "sweep", 256, 2000.0, 10, 20, 20.0, 200.0, 8_000_000),
        # Sixteen mocks of one covariance set through one batched call.
        _case("nodal_batch16_128_f32", "nodal", "sweep", 128, 1000.0, 8, 12, 20.0, 140.0, 600_000, batch=16),
        # Measurement only (no gradient) of a Daubechies-4 reconstruction: the multipoles of a shuffled catalogue.
        _case("nodal_256_d4_forward", "nodal", "forward", 256, 2000.0, 5, 11, 20.0, 200.0, 4_000_001, weights=True,
              order="random", basis="d4"),
        # Particle summation of 1e6 particles, value and gradient.
        _case("particle_128_f32", "particle", "sweep", 128, 1000.0, 10, 15, 20.0, 150.0, 1_000_000),
        # Particle summation in double precision, the value only, of a shuffled weighted catalogue.
        _case("particle_128_f64_forward", "particle", "forward", 128, 1000.0, 6, 9, 20.0, 150.0, 1_000_000, "f64",
              weights=True, order="random"),
        # The largest catalogue: 5e7 weighted particles on 512^3, 20 bins, value and gradient of l <= 1.
        _case("particle_512_f32", "particle", "sweep", 512, 3000.0, 1, 20, 20.0, 200.0, 50_000_000, weights=True),
        # Exact grid summation, value and gradient.
        _case("gamma_128_f32", "gamma", "sweep", 128, 1000.0, 4, 15, 20.0, 150.0, 1_000_000),
        # Exact grid summation on the large grid, the value only.
        _case("gamma_256_f32_forward", "gamma", "forward", 256, 2000.0, 2, 20, 20.0, 200.0, 8_000_000),
        # Exact grid summation on the Daubechies-4 basis, value and gradient.
        _case("gamma_64_d4_f32", "gamma", "sweep", 64, 500.0, 6, 10, 15.0, 100.0, 200_000, basis="d4"),
    ]


def _cost_ms(c):
    """Rough time of a pass, to keep drawn cases below the largest listed one."""
    items = (c["lmax"] + 1) * (c["lmax"] + 2) / 2
    f = 2.0 if c["precision"] == "f64" else 1.0
    e = c["batch"] * c["n"] ** 3 * c["nbins"] / (256.0 ** 3 * 20) * f
    p = c["batch"] * c["particles"] / 5e7 * c["nbins"] / 20 * f
    k = {"sweep": 1.0, "autograd": 1.5, "forward": 0.6, "two_point": 0.0}[c["call"]]
    if c["form"] == "nodal":
        t = 5.5 * e * k
    elif c["form"] == "particle":
        t = 7.0 * e * k + 150.0 * p * (k if k >= 1.0 else 0.4)
    else:
        t = 500.0 * e * (k if k >= 1.0 else 0.4)
    return items * (t + 0.05) + 5.0


def draw(rng):
    """One more case: sizes log-spread over the range of the listed ones, every form, call and precision."""
    while True:
        form = rng.choice(["nodal", "nodal", "particle", "particle", "gamma", "gamma"])
        call = rng.choice(["sweep", "sweep", "sweep", "autograd", "forward"])
        if form == "nodal" and rng.random() < 0.1:
            call = "two_point"   # the two-point function and its line-of-sight multipoles of the same catalogue
        precision = rng.choice(["f32", "f32", "f32", "f64"])
        basis = rng.choice(["b3", "b3", "b3", "d4"])
        if basis == "b3" and precision == "f32" and call == "forward" and rng.random() < 0.3:
            precision = "bf16x3"
        n = rng.choice([16, 32, 32, 64, 64, 128, 128, 256, 256, 512])
        box = round(n * rng.uniform(5.0, 10.0), 1)
        nbins = rng.randint(2, 24)
        lmax = rng.randint(0, 12)
        particles = int(round(n ** 3 * math.exp(rng.uniform(math.log(0.03), math.log(0.6)))))
        batch = rng.choice([1, 1, 1, 2, 3, 5]) if n <= 128 else 1
        c = _case("", form, call, n, box, lmax, nbins, round(box * rng.uniform(0.0, 0.05), 2),
                  round(box * rng.uniform(0.1, 0.24), 2), particles, precision,
                  round(box / n * rng.uniform(0.8, 2.0), 2), rng.random() < 0.5, rng.choice(["cells", "random"]), batch, basis,
                  rng.choice(["shell", "shell", "shell", "thin"]),
                  round(box / n * rng.uniform(1.0, 3.0), 2) if rng.random() < 0.2 else 0.0, rng.random() < 0.15)
        del c["name"]
        if n == 512 and (precision == "f64" or call != "sweep" or nbins > 20 or form == "gamma"):
            continue
        if _cost_ms(c) <= 500.0:
            return c


# -- inputs -----------------------------------------------------------------

def _device():
    return torch.device("cuda", torch.cuda.current_device()) if torch.cuda.is_available() else torch.device("cpu")


def _mock(c, seed, dev):
    """One log-normal catalogue: positions [np, 3] float32 and weights [np] float32 or None."""
    n, box = c["n"], c["box"]
    g = torch.Generator(device=dev).manual_seed(seed)
    noise = torch.fft.rfftn(torch.randn((n, n, n), generator=g, device=dev))
    f = torch.fft.fftfreq(n, d=box / n, device=dev) * (2 * math.pi)
    fz = torch.fft.rfftfreq(n, d=box / n, device=dev) * (2 * math.pi)
    k2 = f[:, None, None] ** 2 + f[None, :, None] ** 2 + fz[None, None, :] ** 2
    k2[0, 0, 0] = 1.0
    spec = k2 ** -0.75 * torch.exp(-k2 * c["smooth"] ** 2)
    spec[0, 0, 0] = 0.0
    field = torch.fft.irfftn(noise * spec.sqrt(), s=(n, n, n))
    del noise, spec, k2
    rho = torch.exp(field / field.std() - 0.5).reshape(-1)
    del field
    # whole weights: their running sum is exact, so a seed always gives the same particles
    edge = torch.cumsum((rho * 2.0 ** 20).to(torch.int64) + 1, 0)
    del rho
    cell = torch.randint(int(edge[-1]), (c["particles"],), generator=g, device=dev)
    if c["order"] == "cells":
        cell = torch.sort(cell)[0]
    cell = torch.searchsorted(edge, cell, right=True)
    del edge
    xyz = torch.stack([cell // (n * n), cell // n % n, cell % n], dim=1)
    del cell
    pos = ((xyz + torch.rand(xyz.shape, generator=g, device=dev, dtype=torch.float64)) * (box / n)).to(torch.float32)
    pos = torch.where(pos >= box, torch.zeros_like(pos), pos).contiguous()
    w = None
    if c["weights"]:
        w = 0.5 + torch.rand(pos.shape[0], generator=g, device=dev)
    return pos, w


def _inputs(c, seed, dev):
    """The catalogues of a batch one after the other, their offsets, and the multipoles' cotangent."""
    mocks = [_mock(c, seed * 1000 + j, dev) for j in range(c["batch"])]
    pos = mocks[0][0] if c["batch"] == 1 else torch.cat([m[0] for m in mocks])
    w = None
    if c["weights"]:
        w = mocks[0][1] if c["batch"] == 1 else torch.cat([m[1] for m in mocks])
    off = [0]
    for m in mocks:
        off.append(off[-1] + m[0].shape[0])
    nb = c["nbins"]
    lam = np.random.default_rng(seed).standard_normal((c["batch"], c["lmax"] + 1, nb, nb))
    return pos, w, off, torch.as_tensor(lam, device=dev)


def _edges(c):
    return np.linspace(c["r_lo"], c["r_hi"], c["nbins"] + 1)


def _radii(c):
    return np.linspace(0.0, c["r_hi"], 3 * c["nbins"] + 1)


def prepare(case, seed):
    dev = _device()
    pos, w, off, lam = _inputs(case, seed, dev)
    plan = mp3.Plan(case["n"], case["box"], case["lmax"], _edges(case), precision=case["precision"],
                    batch=case["batch"], summation=case["form"], binning=case["binning"], smoothing=case["top_hat"],
                    phi_hat=case["phi_hat"], basis=case["basis"])
    autotune.load_tuning(plan)
    if case["call"] == "autograd" and w is None:
        w = torch.ones(pos.shape[0], device=dev)
    return {"call": case["call"], "plan": plan, "pos": pos, "w": w, "off": off, "lam": lam, "radii": _radii(case),
            "ell": min(4, case["lmax"])}


def run(state):
    plan, pos, w, off = state["plan"], state["pos"], state["w"], state["off"]
    if state["call"] == "autograd":
        w = w.detach().requires_grad_()
        zeta = mp3.zeta_from_catalogue(plan, pos, w, off)
        (dw,) = torch.autograd.grad(zeta, w, state["lam"])
        return {"zeta": zeta.detach().to(plan.real_dtype), "dw": dw}
    delta = plan.deposit(pos, w, off)
    if state["call"] == "two_point":
        xi = plan.xi(delta, state["radii"])
        xil = plan.xi_multipoles(delta, state["radii"], state["ell"])
        return {"delta": delta, "xi": xi.to(plan.real_dtype), "xi_ell": xil.to(plan.real_dtype)}
    if state["call"] == "forward":
        zeta = plan.zeta(delta, pos, w, off) if plan.summation == "particle" else plan.zeta(delta)
        return {"delta": delta, "zeta": zeta.to(plan.real_dtype)}
    zeta, ddelta, dw = plan.zeta_value_and_grad(delta, state["lam"], pos, w, off)
    return {"delta": delta, "zeta": zeta.to(plan.real_dtype), "ddelta": ddelta, "dw": dw}


def work(case):
    """Inputs read once, outputs written once; the transforms of every field and the contraction over its points."""
    s = 8 if case["precision"] == "f64" else 4
    n3, nb, B = case["n"] ** 3, case["nbins"], case["batch"]
    items = (case["lmax"] + 1) * (case["lmax"] + 2) / 2
    npart = case["particles"] * B
    grad = case["call"] in ("sweep", "autograd")
    out = B * (case["lmax"] + 1) * nb * nb * s
    nbytes = npart * (12 + (4 if case["weights"] else 0)) + out + (0 if case["call"] == "autograd" else B * n3 * s)
    if grad:
        nbytes += out + npart * s + (0 if case["call"] == "autograd" else B * n3 * s)
    flops = npart * 64 * 2 + B * 5.0 * n3 * math.log2(n3)
    if case["call"] != "two_point":
        points = npart if case["form"] == "particle" else B * n3
        per = 2.0 * nb * (nb + 1)                        # real products of the upper triangle, both parts
        if case["form"] == "particle":
            per += 64 * 4.0 * nb                          # interpolation of every bin
        elif case["form"] == "gamma":
            # points per axis and cell: half the dimension of the splines of the product (degree 9, C^2) rounded
            # up for the B-spline; the band of the connection coefficients for Daubechies-4
            q = 4 if case["basis"] == "b3" else 3
            per = q ** 3 * (per + 8 * 4.0 * nb)
        flops += items * (B * nb * 5.0 * n3 * math.log2(n3) + points * per)
        if grad:
            flops += items * (B * nb * 5.0 * n3 * math.log2(n3) + points * (per - 2.0 * nb * (nb + 1)))
    return {"bytes": float(nbytes), "flops": float(flops)}


# -- the same outputs in 64 bits, from the estimator's definitions ------------

_C = torch.complex128


def _sph_jn(l, x):
    """j_l(x) for x >= 0: upward recurrence for x > l + 1, the power series below."""
    big = x > l + 1.0
    xb = torch.where(big, x, torch.full_like(x, l + 2.0))
    a, b = torch.sin(xb) / xb, torch.sin(xb) / xb ** 2 - torch.cos(xb) / xb
    for k in range(1, l + 1):
        a, b = b, (2 * k + 1) / xb * b - a
    xs = torch.where(big, torch.zeros_like(x), x)
    t = torch.ones_like(x)
    for k in range(1, l + 1):
        t = t * xs / (2 * k + 1)
    s = t.clone()
    for k in range(1, 60):
        t = t * (-0.5 * xs * xs) / (k * (2 * l + 2 * k + 1))
        s += t
    return torch.where(big, a, s)


def _top_hat(x):
    big = x > 0.02
    xb = torch.where(big, x, torch.ones_like(x))
    return torch.where(big, 3 * (torch.sin(xb) - xb * torch.cos(xb)) / xb ** 3, 1 - x * x / 10 + x ** 4 / 280)


def _radial(c, l, dev):
    """The radial window of every |q|^2 and bin, [3 (n/2)^2 + 1, nbins]."""
    k = torch.sqrt(torch.arange(3 * (c["n"] // 2) ** 2 + 1, dtype=torch.float64, device=dev)) * (2 * math.pi / c["box"])
    e = _edges(c)
    cols = []
    x, wq = np.polynomial.legendre.leggauss(48)
    for b in range(c["nbins"]):
        r0, r1 = e[b], e[b + 1]
        if c["binning"] == "thin":
            cols.append(_sph_jn(l, k * (0.5 * (r0 + r1))))
            continue
        r = torch.as_tensor(0.5 * (r1 - r0) * x + 0.5 * (r0 + r1), device=dev)
        wr = torch.as_tensor(0.5 * (r1 - r0) * wq, device=dev) * r * r * (3.0 / (r1 ** 3 - r0 ** 3))
        cols.append(_sph_jn(l, k[:, None] * r[None, :]) @ wr)
    out = torch.stack(cols, dim=1)
    return out * _top_hat(k * c["top_hat"])[:, None] if c["top_hat"] > 0 else out


_H4 = np.array([1 + math.sqrt(3), 3 + math.sqrt(3), 3 - math.sqrt(3), 1 - math.sqrt(3)]) / (4 * math.sqrt(2))


def _d4_table():
    """The Daubechies-4 scaling function at i / 1024 on [0, 3], by the two-scale relation."""
    v = {0: 0.0, 1: (1 + math.sqrt(3)) / 2, 2: (1 - math.sqrt(3)) / 2, 3: 0.0}
    tab = np.array([v[i] for i in range(4)])
    for level in range(1, 11):
        size = 3 * 2 ** level + 1
        new = np.zeros(size)
        half = 2 ** (level - 1)
        for i in range(size):
            if i % 2 == 0:
                new[i] = tab[i // 2]
            else:   # phi(x) = sqrt2 sum_k h_k phi(2x - k), 2x = i / 2^(level-1)
                new[i] = math.sqrt(2) * sum(_H4[k] * tab[i - k * half] for k in range(4)
                                            if 0 <= i - k * half < len(tab))
        tab = new
    return tab


def _d4_acf(tab):
    """int phi(x) phi(x - s) dx of the table's linear interpolant, s = 0 .. 3."""
    out = []
    for s in range(4):
        a, b = tab[s * 1024:], tab[:len(tab) - s * 1024]
        out.append(float(np.sum(2 * a[:-1] * b[:-1] + 2 * a[1:] * b[1:] + a[:-1] * b[1:] + a[1:] * b[:-1]) / 6 / 1024))
    return out


def _d4_connection():
    """gamma(s, t) = int phi(x) phi(x - s) phi(x - t) dx, s, t = -2 .. 2, from the two-scale relation."""
    idx = [(s, t) for s in range(-2, 3) for t in range(-2, 3) if abs(s - t) <= 2]
    at = {p: i for i, p in enumerate(idx)}
    M = np.zeros((len(idx), len(idx)))
    for (s, t), i in at.items():
        for k in range(4):
            for a in range(4):
                for b in range(4):
                    j = at.get((2 * s + a - k, 2 * t + b - k))
                    if j is not None:
                        M[i, j] += math.sqrt(2) * _H4[k] * _H4[a] * _H4[b]
    A = np.vstack([M - np.eye(len(idx)), np.ones(len(idx))])
    sol = np.linalg.lstsq(A, np.r_[np.zeros(len(idx)), 1.0], rcond=None)[0]
    g = np.zeros((5, 5))
    for (s, t), i in at.items():
        g[s + 2, t + 2] = sol[i]
    return 0.5 * (g + g.T)


def _taps(c, pos, dev):
    """First node and four weights per axis of every particle."""
    n = c["n"]
    u = torch.remainder(pos.to(torch.float64) * (n / c["box"]), float(n))
    cell = torch.floor(u)
    f = u - cell
    cell = cell.to(torch.int64) % n
    if c["basis"] == "b3":
        g = 1 - f
        w = [g ** 3 / 6, 2 / 3 - f * f + f ** 3 / 2, 2 / 3 - g * g + g ** 3 / 2, f ** 3 / 6]
    else:
        tab = torch.as_tensor(_d4_table(), device=dev)
        w = []
        for o in (-1, 0, 1):   # node cell + o carries phi(u - node + 1)
            x = (f - o + 1) * 1024
            i = torch.clamp(torch.floor(x).to(torch.int64), 0, 3071)
            w.append(tab[i] + (tab[i + 1] - tab[i]) * (x - i))
        w.append(torch.zeros_like(f))
    return (cell - 1) % n, torch.stack(w, dim=-1)


def _each_tap(c, cell, wt):
    n = c["n"]
    for i in range(4):
        for j in range(4):
            for k in range(4):
                at = (((cell[:, 0] + i) % n) * n + (cell[:, 1] + j) % n) * n + (cell[:, 2] + k) % n
                yield at, wt[:, 0, i] * wt[:, 1, j] * wt[:, 2, k]


def _rule(c, dev):
    """Points per axis of the grid summation: (transform of the fields' filter, of the primary's, weight)."""
    q = torch.fft.fftfreq(c["n"], d=1.0 / c["n"], device=dev, dtype=torch.float64)
    one = torch.ones(c["n"], dtype=_C, device=dev)

    def factor(v, first):
        return sum(float(a) * torch.exp(2j * math.pi * (first + o) * q / c["n"]) for o, a in enumerate(v))

    if c["form"] != "gamma":
        return [(one, one, 1.0)]
    if c["basis"] == "d4":
        val, vec = np.linalg.eigh(_d4_connection())
        return [(factor(vec[:, s], -2), one, float(val[s])) for s in range(5)]
    out = []
    for x, w in zip(*np.polynomial.legendre.leggauss(5)):
        f = 0.5 * (x + 1)
        g = 1 - f
        v = [g ** 3 / 6, 2 / 3 - f * f + f ** 3 / 2, 2 / 3 - g * g + g ** 3 / 2, f ** 3 / 6]
        out.append((factor(v, -1), factor(v, -1), 0.5 * float(w)))
    return out


def _legendre_lm(l, m, mu):
    """Orthonormal associated Legendre function of cos(theta), without the factor sin(theta)^m."""
    p = torch.ones_like(mu) * math.sqrt(1 / (4 * math.pi))
    for k in range(1, m + 1):
        p = -p * math.sqrt((2 * k + 1) / (2 * k))
    if l == m:
        return p
    prev, p = p, math.sqrt(2 * m + 3) * mu * p
    for k in range(m + 2, l + 1):
        a = math.sqrt((4 * k * k - 1) / (k * k - m * m))
        b = math.sqrt(((k - 1) ** 2 - m * m) / (4 * (k - 1) ** 2 - 1))
        prev, p = p, a * (mu * p - b * prev)
    return p


class _Grid:
    """Wavenumbers and windows of one case."""

    def __init__(self, c, dev):
        n = c["n"]
        q = torch.fft.fftfreq(n, d=1.0 / n, device=dev, dtype=torch.float64)
        qx, qy, qz = q[:, None, None], q[None, :, None], q[None, None, :]
        self.q2 = (qx * qx + qy * qy + qz * qz).to(torch.int64)
        qq = torch.sqrt(self.q2.to(torch.float64))
        self.mu = qz / torch.where(qq > 0, qq, torch.ones_like(qq))
        self.qq = qq
        self.rho = torch.complex(qx + 0 * qy, -(qy + 0 * qx)) / torch.where(qq > 0, qq, torch.ones_like(qq))
        keep = (q != -(n // 2)).to(torch.float64)
        self.keep = keep[:, None, None] * keep[None, :, None] * keep[None, None, :]
        self.wth = _top_hat(qq * (2 * math.pi / c["box"] * c["top_hat"]))
        self.phi = None
        if c["phi_hat"]:
            if c["basis"] == "b3":
                p = torch.sinc(q / n) ** 8
            else:
                p = torch.ones_like(q)
                for j in range(1, 65):
                    xi = 2 * math.pi * q / n / 2.0 ** j
                    p = p * torch.cos(xi / 2) ** 4 * (1 + 2 * torch.sin(xi / 2) ** 2)
            self.phi = p[:, None, None] * p[None, :, None] * p[None, None, :]
            self.keep = self.keep * self.phi
        self.n = n

    def angular(self, l, m):
        y = _legendre_lm(l, m, self.mu) * self.rho ** m * (1j ** l) * self.keep
        y[0, 0, 0] = (1 if l == 0 else 0) / math.sqrt(4 * math.pi)
        return y


def _outer(a, b, z):
    return a[:, None, None] * b[None, :, None] * z[None, None, :]


def _gram(a, b):
    """sum_x Re a_i(x) conj(b_j(x)) of two [bins, points] fields, in blocks of points."""
    k = a.shape[1]
    parts = max(1, min(256, k // 4096))
    while k % parts:
        parts -= 1
    u = torch.view_as_real(a).reshape(a.shape[0], parts, -1).transpose(0, 1).contiguous()
    v = torch.view_as_real(b).reshape(b.shape[0], parts, -1).permute(1, 2, 0).contiguous()
    return torch.bmm(u, v).sum(0)


def _one_mock(c, pos, w, lam, dev):
    n, nb, L = c["n"], c["nbins"], c["lmax"]
    n3, four_pi = n ** 3, 4 * math.pi
    grad = c["call"] in ("sweep", "autograd")
    particle = c["form"] == "particle"
    w = torch.ones(pos.shape[0], dtype=torch.float64, device=dev) if w is None else w.to(torch.float64)
    W = w.sum()
    cell, wt = _taps(c, pos, dev)
    eps = torch.zeros(n3, dtype=torch.float64, device=dev)
    for at, t in _each_tap(c, cell, wt):
        eps.index_add_(0, at, t * w)
    delta = (eps * (n3 / W) - 1).reshape(n, n, n)
    del eps
    dhat = torch.fft.fftn(delta)
    g = _Grid(c, dev)
    if c["call"] == "two_point":
        r = torch.as_tensor(_radii(c), device=dev)
        size = 3 * (n // 2) ** 2 + 1
        k = torch.sqrt(torch.arange(size, dtype=torch.float64, device=dev)) * (2 * math.pi / c["box"])
        wk = (_top_hat(k * c["top_hat"]) ** 2 if c["top_hat"] > 0 else torch.ones_like(k))
        xil = []
        p0, p1 = torch.ones_like(g.mu), g.mu
        for l in range(min(4, L) + 1):
            hist = torch.zeros(size, dtype=torch.float64, device=dev)
            hist.index_add_(0, g.q2.reshape(-1), (dhat.abs() ** 2 * g.keep * p0).reshape(-1))
            if l > 0:
                hist[0] = 0
            kernel = torch.stack([_sph_jn(l, k * x) for x in r]) * ((2 * l + 1) * (1j ** l).real)
            xil.append(kernel @ (hist * wk) / n3 ** 2)
            p0, p1 = p1, ((2 * l + 3) * g.mu * p1 - (l + 1) * p0) / (l + 2)
        return {"delta": delta, "xi": xil[0], "xi_ell": torch.stack(xil)}
    prim_hat = dhat * g.wth if c["top_hat"] > 0 and not particle else dhat
    rule = _rule(c, dev)
    zeta = torch.zeros((L + 1, nb, nb), dtype=torch.float64, device=dev)
    G = torch.zeros((n, n, n), dtype=_C, device=dev)
    direct = torch.zeros((n, n, n), dtype=_C, device=dev)      # transform of the primary's share
    FJ = torch.zeros(pos.shape[0], dtype=torch.float64, device=dev)
    acf = [2416 / 5040, 1191 / 5040, 120 / 5040, 1 / 5040] if c["basis"] == "b3" else _d4_acf(_d4_table())
    th = torch.fft.fftfreq(n, device=dev, dtype=torch.float64) * (2 * math.pi)
    ax = acf[0] + 2 * sum(acf[s] * torch.cos(s * th) for s in (1, 2, 3))
    mean_w = _outer(ax, ax, ax) * (g.keep if g.phi is None else g.keep * g.phi)
    h2 = torch.zeros(3 * (n // 2) ** 2 + 1, dtype=torch.float64, device=dev)
    P = torch.zeros_like(h2)
    if particle:
        P.index_add_(0, g.q2.reshape(-1), (dhat.abs() ** 2 * mean_w).reshape(-1))
    for l in range(L + 1):
        jr = _radial(c, l, dev)
        ls = 0.5 * (lam[l] + lam[l].T)
        jg = jr.T.contiguous()[:, g.q2.reshape(-1)].reshape(nb, n, n, n)
        for m in range(l + 1):
            wm = 1.0 if m == 0 else 2.0
            K = jg * g.angular(l, m)
            if l:
                K[:, 0, 0, 0] = 0
            F = K * dhat
            if not grad:
                del K
            if particle:
                a = torch.fft.ifftn(F, dim=(1, 2, 3)).reshape(nb, n3).T.contiguous()
                del F
                at_p = torch.zeros((pos.shape[0], nb), dtype=_C, device=dev)
                for at, t in _each_tap(c, cell, wt):
                    at_p += a[at] * t[:, None]
                ri = torch.view_as_real(at_p)
                for part in (ri[..., 0].contiguous(), ri[..., 1].contiguous()):
                    zeta[l] += wm * four_pi / W * (part.T @ (part * w[:, None]))
                if grad:
                    u = at_p @ ls.to(_C)
                    FJ += wm * (at_p * u.conj()).real.sum(1)
                    s = torch.view_as_real(u.conj() * (w * (n3 / W))[:, None]).reshape(-1, 2 * nb)
                    src = torch.zeros((n3, 2 * nb), dtype=torch.float64, device=dev)
                    for at, t in _each_tap(c, cell, wt):
                        src.index_add_(0, at, s * t[:, None])
                    src = torch.view_as_complex(src.reshape(n3, nb, 2)).T.contiguous().reshape(nb, n, n, n)
                    G += wm * (K * torch.fft.ifftn(src, dim=(1, 2, 3))).sum(0)
                continue
            cx = torch.zeros_like(F) if grad and len(rule) > 1 else None
            for fx, px, wx in rule:
                Fx = torch.fft.ifft(F * fx[:, None, None], dim=1)
                cy = torch.zeros_like(F) if cx is not None else None
                for fy, py, wy in rule:
                    Fy = torch.fft.ifft(Fx * fy[:, None], dim=2)
                    cz = torch.zeros_like(F) if cx is not None else None
                    for fz, pz, wz in rule:
                        a = torch.fft.ifft(Fy * fz, dim=3)
                        pf = _outer(px, py, pz)
                        prim = torch.fft.ifftn(prim_hat * pf).real * (wx * wy * wz)
                        pa = (a * prim).reshape(nb, n3)
                        zeta[l] += wm * four_pi / n3 * _gram(a.reshape(nb, n3), pa)
                        if not grad:
                            continue
                        ua = (ls @ torch.view_as_real(a).reshape(nb, -1)).reshape(nb, n, n, n, 2)
                        ua = torch.view_as_complex(ua)
                        share = (a * ua.conj()).real.sum(0) * (wm * wx * wy * wz)
                        direct += pf.conj() * torch.fft.fftn(share)
                        src = torch.fft.ifft(ua.conj() * prim, dim=3)
                        cz = src if cz is None else cz.add_(src * fz)
                    if grad:
                        cz = torch.fft.ifft(cz, dim=2)
                        cy = cz if cy is None else cy.add_(cz * fy[:, None])
                if grad:
                    cy = torch.fft.ifft(cy, dim=1)
                    cx = cy if cx is None else cx.add_(cy * fx[:, None, None])
            if grad:
                G += wm * (K * cx).sum(0)
        if particle:
            zeta[l] -= (2 * l + 1) / n3 ** 2 * (jr.T @ (jr * P[:, None]))
            h2 += (2 * l + 1) * (jr * (jr @ ls)).sum(1)
    if not grad:
        return {"delta": delta, "zeta": zeta}
    if particle:
        G -= mean_w * h2[g.q2] * dhat.conj() / (four_pi * n3)
    ddelta = 2 * torch.fft.fftn(G).real * (four_pi / n3)
    if not particle:
        if c["top_hat"] > 0:
            direct = direct * g.wth
        ddelta = ddelta + torch.fft.ifftn(direct).real * (four_pi / n3)
    gi = torch.zeros(pos.shape[0], dtype=torch.float64, device=dev)
    flat = ddelta.reshape(-1)
    for at, t in _each_tap(c, cell, wt):
        gi += flat[at] * t
    dw = (n3 / W) * (gi - ((1 + delta) * ddelta).sum() / n3)
    if particle:
        dw = dw + four_pi * (FJ / W - (w * FJ).sum() / W ** 2)
    if c["call"] == "autograd":
        return {"zeta": zeta, "dw": dw}
    return {"delta": delta, "zeta": zeta, "ddelta": ddelta, "dw": dw}


def _exact_seconds(c):
    """Rough time of exact()."""
    items = (c["lmax"] + 1) * (c["lmax"] + 2) / 2 if c["call"] != "two_point" else 1
    e = c["batch"] * items * c["n"] ** 3 * c["nbins"] / (256.0 ** 3 * 20)
    p = c["batch"] * items * c["particles"] * c["nbins"] / (1e6 * 15)
    grad = 2.0 if c["call"] in ("sweep", "autograd") else 1.0
    if c["form"] == "particle":
        return grad * (0.1 * e + 0.1 * p)
    return grad * e * (0.08 if c["form"] == "nodal" else 125 * 0.02)


def exact(case, seed):
    if case["n"] > 256 or _exact_seconds(case) > 20.0:
        return None
    dev = _device()
    pos, w, off, lam = _inputs(case, seed, dev)
    out = []
    for j in range(case["batch"]):
        s = slice(off[j], off[j + 1])
        out.append(_one_mock(case, pos[s], None if w is None else w[s], lam[j], dev))
    per_particle = ("dw",)
    return {k: torch.cat([o[k] for o in out]) if k in per_particle else torch.stack([o[k] for o in out])
            for k in out[0]}
