"""Performance cases of the registration path: what its users run, through the package's entry points.

A case is a dict with

  op      "operator"   K f or L f (``Registration.apply_operator``): the metric operator by itself
          "shoot"      a forward geodesic with its warp: J_1, u_1, v_1, the energy and det(I + D u_1)
          "gradient"   energy and V-gradient at v0: trajectory store, final conditions, adjoint sweep
          "hessvec"    Gauss-Newton Hessian-vector product at a linearization (the inner step of CG)
          "newton"     the same on the full Newton Hessian, from v0 (linearization included)
          "autograd"   ``shoot_image`` inside a torch loss: forward and backward
          "pde"        PDE-LDDMM: gradient at v and the Hessian product at that linearization
          "solve"      a whole Gauss-Newton-Krylov solve of a few outer iterations
  n0, n1, n2, nt       grid (products of 2, 3, 5, 7) and time steps
  dtype                "f32" or "f64": the element type of every field
  ...                  options of the op, named below

Images, velocities and directions are drawn on the GPU from the seed alone: phantoms of an ellipsoidal
shell and Gaussian blobs with their noise, and band-limited velocities of a few per cent of the box, as
the repository's own workloads have them.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_1807_04638_amd import Registration
from paper_1807_04638_amd.autograd import shoot_image

ALPHA, POWER, SIGMA2 = 0.0025, 2, 1.0
DEV = "cuda:0"
_DTYPE = {"f32": torch.float32, "f64": torch.float64}


def _case(name, op, n, nt, dtype, **more):
    return {"name": name, "op": op, "n0": n[0], "n1": n[1], "n2": n[2], "nt": nt, "dtype": dtype, **more}


def listed():
    return [
        # one metric-operator call on a coarse pyramid level: latency and launches
        _case("operator_32_f32", "operator", (32, 32, 32), 10, "f32", L=False, ncomp=3),
        # the metric operator on the grid that the brain volumes are resampled to (x1 = 2 3 5 7), double
        _case("operator_180x210x180_f64", "operator", (180, 210, 180), 10, "f64", L=True, ncomp=3),
        # applying a found registration to an image on a coarse level
        _case("shoot_64_f32", "shoot", (64, 64, 64), 10, "f32"),
        # the gradient of the benchmark's pair
        _case("gradient_128_f32", "gradient", (128, 128, 128), 10, "f32", every=0),
        # the Hessian product of the benchmark's pair, replayed from a graph as CG does
        _case("hessvec_128_f32", "hessvec", (128, 128, 128), 10, "f32", graph=True),
        # the precision workload's grid in double
        _case("hessvec_180x216x180_f64", "hessvec", (180, 216, 180), 16, "f64", graph=False),
        # the resampling grid of the brain volumes in single precision
        _case("hessvec_180x210x180_f32", "hessvec", (180, 210, 180), 10, "f32", graph=False),
        # the Newton product of a mid-size pair of the batch
        _case("newton_96_f32", "newton", (96, 96, 96), 10, "f32"),
        # a warped template inside a torch loss on a cropped, anisotropic volume, double
        _case("autograd_60x84x70_f64", "autograd", (60, 84, 70), 10, "f64"),
        # the comparison method with one velocity field per time point
        _case("pde_128_f32", "pde", (128, 128, 128), 10, "f32", stationary=False),
        # the largest volume, its trajectory checkpointed
        _case("gradient_256_f32", "gradient", (256, 256, 256), 32, "f32", every=4),
        # a whole registration on the plain-method grid (32^3): hundreds of small launches
        _case("solve_32_f32", "solve", (32, 32, 32), 10, "f32", iters=2, cg=8),
    ]


# lengths a grid may have: products of 2, 3, 5, 7
_LENGTHS = [n for n in range(16, 257) if all(p in (2, 3, 5, 7) for p in range(2, n + 1)
                                             if n % p == 0 and all(p % q for q in range(2, p)))]
# passes over the grid that one time step of an op makes, in gradients
_WEIGHT = {"operator": 0.03, "shoot": 0.5, "gradient": 1.0, "hessvec": 1.0, "newton": 3.2, "autograd": 1.0,
           "pde": 1.2, "solve": 12.0}


def draw(rng):
    op = rng.choice(["operator", "shoot", "gradient", "hessvec", "hessvec", "newton", "autograd", "pde", "solve"])
    dtype = rng.choice(["f32", "f32", "f64"])
    side = math.exp(rng.uniform(math.log(20.0), math.log(240.0)))
    n = []
    for d in range(3):
        want = side * rng.uniform(0.75, 1.3)
        ok = [m for m in _LENGTHS if d < 2 or m % 2 == 0]
        n.append(min(ok, key=lambda m: abs(m - want)))
    nt = rng.choice([8, 10, 12, 16])
    # no more than the largest listed case: 256^3, 32 steps, a checkpointed gradient in single precision
    budget = 256.0**3 * 32 * (0.5 if op in ("newton", "pde", "solve") else 1.0)
    while n[0] * n[1] * n[2] * nt * _WEIGHT[op] * (2.0 if dtype == "f64" else 1.0) > budget:
        n = [max([m for m in _LENGTHS if m < x and (d < 2 or m % 2 == 0)] or [16]) for d, x in enumerate(n)]
    case = _case("", op, n, nt, dtype)
    del case["name"]
    if op == "operator":
        case.update(L=rng.random() < 0.4, ncomp=rng.choice([1, 3]))
    elif op == "gradient":
        case.update(every=rng.choice([0, 0, 4]))
    elif op == "hessvec":
        case.update(graph=rng.random() < 0.5)
    elif op == "pde":
        case.update(stationary=rng.random() < 0.5)
    elif op == "solve":
        case.update(iters=2, cg=rng.choice([4, 8]))
    return case


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _band_limited(n, gen, ncomp):
    """Low-pass filtered noise (ncomp, n0, n1, n2) in double: exp(-|k|^2 / (2 kc^2)), kc = N / 16."""
    kc = max(1.0, min(n) / 16.0)
    k2 = _ksq(n)
    f = torch.randn((ncomp,) + n, generator=gen, device=DEV, dtype=torch.float64)
    for c in range(ncomp):
        f[c] = torch.fft.irfftn(torch.fft.rfftn(f[c]) * torch.exp(-0.5 * k2 / kc**2), s=n)
    return f


def _velocity(n, gen, share):
    """Band-limited velocity whose largest displacement is `share` of the box's shortest side."""
    v = _band_limited(n, gen, 3)
    return v * (share * 2.0 * math.pi / v.square().sum(0).max().sqrt())


def _pair(n, seed):
    """A template and a target of the same subject's kind: shell and blobs, the target's moved and noisy."""
    r = np.random.default_rng(seed)
    x = [torch.arange(m, device=DEV, dtype=torch.float64) for m in n]
    semi = [0.38 * n[0], 0.42 * n[1], 0.36 * n[2]]
    rho = sum(((x[d] - n[d] / 2.0) / semi[d]).square().reshape([-1 if e == d else 1 for e in range(3)])
              for d in range(3)).sqrt()
    shell = 0.5 / (1.0 + torch.exp((rho - 0.95).abs() * 60.0 - 3.0))
    del rho
    images = [shell, shell.clone()]
    for _ in range(16):
        at = r.uniform(-0.45, 0.45, 3)
        sig = r.uniform(0.03, 0.09, 3)
        amp = r.choice([0.2, 0.5, 0.8])
        for img, move in zip(images, (np.zeros(3), r.normal(0.0, 0.015, 3))):
            e = [torch.exp(-0.5 * ((x[d] / n[d] - 0.5 - at[d] * semi[d] / n[d] * 2.0 * 0.9 - move[d]) / sig[d]).square())
                 for d in range(3)]
            img += amp * e[0][:, None, None] * e[1][None, :, None] * e[2][None, None, :]
    I0, I1 = (img.clamp_(0.0, 1.0) for img in images)
    I1 += 0.01 * torch.randn(n, generator=_gen(seed + 7), device=DEV, dtype=torch.float64)
    return I0, I1


def _inputs(case, seed):
    """Every array the case's call takes, in the case's type (``exact`` starts from the same ones)."""
    n = (case["n0"], case["n1"], case["n2"])
    dt = _DTYPE[case["dtype"]]
    op = case["op"]
    gen = _gen(seed)
    d = {}
    if op == "operator":
        f = _band_limited(n, gen, case["ncomp"])
        f += 0.01 * torch.randn(f.shape, generator=gen, device=DEV, dtype=torch.float64)
        d["f"] = f if case["ncomp"] == 3 else f[0]
    else:
        d["I0"], d["I1"] = _pair(n, seed)
        if op == "pde" and not case["stationary"]:
            d["v0"] = torch.stack([_velocity(n, gen, 0.03) for _ in range(2)])
            t = torch.linspace(0.0, 1.0, case["nt"] + 1, device=DEV, dtype=torch.float64).reshape(-1, 1, 1, 1, 1)
            d["v0"] = (1.0 - t) * d["v0"][0] + t * d["v0"][1]
            w = _velocity(n, gen, 0.01)
            d["dv"] = (1.0 - 0.5 * t) * w
        elif op != "solve":
            d["v0"] = _velocity(n, gen, 0.03)
            if op in ("hessvec", "newton", "pde"):
                d["dv"] = _velocity(n, gen, 0.01)
    return {k: x.to(dt).contiguous() for k, x in d.items()}


# --------------------------------------------------------------------------
# What a program keeps, and one pass
# --------------------------------------------------------------------------
_stream = None


def _side_stream():
    """The stream of a program that replays graphs (one for all of its contexts)."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream(device=DEV)
    return _stream


def prepare(case, seed):
    op = case["op"]
    st = {"case": case}
    graph = bool(case.get("graph"))
    with torch.cuda.stream(_side_stream() if graph else torch.cuda.current_stream()):
        st.update(_inputs(case, seed))
        R = Registration((case["n0"], case["n1"], case["n2"]), case["nt"], ALPHA, POWER, SIGMA2,
                         dtype=_DTYPE[case["dtype"]], device=DEV, checkpoint_every=case.get("every", 0))
        st["R"] = R
        if op != "operator":
            R.set_images(st["I0"], st["I1"])
        if op == "hessvec":
            if graph:
                R.set_option("exec.graph", 1)
            R.linearize(st["v0"])
            st["hv"] = torch.empty_like(st["dv"])
    torch.cuda.synchronize()
    return st


def run(state):
    case, R, op = state["case"], state["R"], state["case"]["op"]
    if op == "operator":
        return (R.apply_L if case["L"] else R.apply_K)(state["f"])
    if op == "shoot":
        r = R.shoot(state["v0"], energy=True)
        det, lo, hi = R.jacobian_det(r["u1"])
        return {"J1": r["J1"], "u1": r["u1"], "v1": r["v1"], "energy": r["energy"], "det": det, "det_min": lo,
                "det_max": hi}
    if op == "gradient":
        g, e = R.gradient(state["v0"])
        return {"g": g, "energy": e}
    if op == "hessvec":
        if not case["graph"]:
            return R.hessvec(state["dv"])
        with torch.cuda.stream(_side_stream()):
            return R.hessvec(state["dv"], out=state["hv"])
    if op == "newton":
        return R.hessvec(state["dv"], v0=state["v0"], newton=True)
    if op == "autograd":
        v0 = state["v0"].detach().requires_grad_(True)
        J1 = shoot_image(R, v0)
        (0.5 * (J1 - state["I1"]).square().sum()).backward()
        return {"J1": J1.detach(), "grad": v0.grad}
    if op == "pde":
        g, e = R.pde_gradient(state["v0"], stationary=case["stationary"])
        return {"g": g, "energy": e, "hv": R.pde_hessvec(state["dv"], stationary=case["stationary"])}
    v = torch.zeros((3,) + R.n, dtype=R.dtype, device=R.device)
    t = R.gn_solve(v, gn_iters=case["iters"], cg_iters=case["cg"])
    return {"v0": v, "energy": [t.log[0]["E"], t.report["E_final"]], "mse_rel": t.report["mse_rel_final"]}


def work(case):
    """One time step of one sweep reads four coefficient fields (v, mu at both Heun stages) and makes two
    K applications and two stencil stages; a field is read or written once by each that needs it."""
    n = case["n0"] * case["n1"] * case["n2"]
    V = 3 * n * (4 if case["dtype"] == "f32" else 8)
    fft = 2 * 3 * 2.5 * n * math.log2(n)  # forward and inverse real transforms of a vector field
    op, nt = case["op"], case["nt"]
    shoot = {"bytes": (4 + 2) * V * nt, "flops": (2 * fft + 2 * 60 * n + 250 * n) * nt}
    sweep = {"bytes": (4 + 2) * V * nt, "flops": (2 * fft + 2 * 180 * n) * nt}
    if op == "operator":
        c = case["ncomp"] / 3.0
        return {"bytes": 2 * V * c, "flops": fft * c}
    if op == "pde":
        m = 1 if case["stationary"] else nt + 1
        per = V / 3 * nt
        return {"bytes": 4 * V * m + 2 * (4 * per + 3 * per + V * (nt if m > 1 else 1)),
                "flops": 2 * m * fft + 4 * 250 * n * nt}
    s, b = {"shoot": (1, 0), "gradient": (1, 1), "hessvec": (0, 2), "newton": (1, 3.7), "autograd": (1, 1),
            "solve": (1 + case.get("iters", 0), case.get("iters", 0) * (1 + 2 * 2))}[op]
    return {k: s * shoot[k] + b * sweep[k] for k in shoot}


# --------------------------------------------------------------------------
# The same in 64 bits by plain torch
# --------------------------------------------------------------------------
def _ksq(n):
    k = [torch.fft.fftfreq(m, 1.0 / m, device=DEV, dtype=torch.float64) for m in n[:2]]
    k.append(torch.fft.rfftfreq(n[2], 1.0 / n[2], device=DEV, dtype=torch.float64))
    return k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + k[2][None, None, :] ** 2


class _Exact:
    """The method on the grid, one whole-array expression per equation."""

    def __init__(self, case, inputs):
        self.n = (case["n0"], case["n1"], case["n2"])
        self.nt = case["nt"]
        self.dt = 1.0 / self.nt
        self.h = [2.0 * math.pi / m for m in self.n]
        self.cell = self.h[0] * self.h[1] * self.h[2]
        self.symbol = (1.0 + ALPHA * _ksq(self.n)) ** POWER
        self.I0, self.I1 = inputs.get("I0"), inputs.get("I1")
        self.strides = [self.n[1] * self.n[2], self.n[2], 1]

    def _spectral(self, f, mult):
        if f.dim() == 3:
            return torch.fft.irfftn(torch.fft.rfftn(f) * mult, s=self.n)
        return torch.stack([torch.fft.irfftn(torch.fft.rfftn(x) * mult, s=self.n) for x in f])

    def L(self, f):
        return self._spectral(f, self.symbol)

    def K(self, f):
        return self._spectral(f, 1.0 / self.symbol)

    def d(self, f, e):
        return (torch.roll(f, -1, e) - torch.roll(f, 1, e)) / (2.0 * self.h[e])

    def grad(self, f):
        return torch.stack([self.d(f, e) for e in range(3)])

    def inner(self, a, b):
        return self.cell * float((a * b).sum())

    def ad(self, v, w):
        return torch.stack([sum(self.d(v[c], e) * w[e] - self.d(w[c], e) * v[e] for e in range(3)) for c in range(3)])

    def ad_star(self, v, m):
        return torch.stack([sum(self.d(v[e], c) * m[e] + self.d(m[c] * v[e], e) for e in range(3)) for c in range(3)])

    # periodic trilinear interpolation of f (..., n0, n1, n2) at x + q, q in voxels
    def at(self, f, q):
        lo, t = [], []
        for e in range(3):
            fl = torch.floor(q[e])
            t.append(q[e] - fl)
            i = torch.arange(self.n[e], device=DEV).reshape([-1 if a == e else 1 for a in range(3)])
            lo.append(i + fl.to(torch.int64))
        flat = f.reshape(-1, self.n[0] * self.n[1] * self.n[2])
        out = torch.zeros((flat.shape[0],) + self.n, device=DEV, dtype=torch.float64)
        for corner in range(8):
            idx, w = 0, 1.0
            for e in range(3):
                up = corner >> e & 1
                idx = idx + torch.remainder(lo[e] + up, self.n[e]) * self.strides[e]
                w = w * (t[e] if up else 1.0 - t[e])
            for c in range(flat.shape[0]):
                out[c] += w * flat[c][idx]
        return out[0] if f.dim() == 3 else out

    def vox(self, v):
        return [v[e] / self.h[e] for e in range(3)]

    def foot(self, v_old, v_new):  # displacement of the backward characteristic's foot
        return -0.5 * self.dt * (v_new + self.at(v_old, self.vox(-self.dt * v_new)))

    def shoot(self, v0):
        mu, v = self.L(v0), v0
        u = torch.zeros_like(v0)
        self.path = []
        for _ in range(self.nt):
            ms = mu - self.dt * self.ad_star(v, mu)
            vs = self.K(ms)
            m2 = 0.5 * mu + 0.5 * (ms - self.dt * self.ad_star(vs, ms))
            v2 = self.K(m2)
            x = self.foot(v, v2)
            u = self.at(u, self.vox(x)) + x
            self.path.append((mu, v, ms, vs))
            mu, v = m2, v2
        self.J1 = self.at(self.I0, self.vox(u))
        self.res = self.J1 - self.I1
        self.G = self.grad(self.J1)
        self.E = self.inner(self.path[0][0], v0) + self.inner(self.res, self.res) / SIGMA2
        return u, v

    def backward(self, U, keep=None):
        w = torch.zeros_like(U)
        for mu, v, ms, vs in reversed(self.path):
            Us = U + self.dt * self.ad_star(vs, U)
            ws = w + self.dt * (self.K(U + self.ad_star(w, ms)) - self.ad(vs, w))
            if keep is not None:
                keep.append((U, w, Us, ws))
            U2 = 0.5 * U + 0.5 * (Us + self.dt * self.ad_star(v, Us))
            w = 0.5 * w + 0.5 * (ws + self.dt * (self.K(Us + self.ad_star(ws, mu)) - self.ad(v, ws)))
            U = U2
        return w

    def gradient(self, v0):
        return 2.0 * v0 + self.backward(-2.0 / SIGMA2 * self.res * self.G)

    def tangent(self, dv, keep=None):
        X, m = torch.zeros_like(dv), self.L(dv)
        for mu, v, ms, vs in self.path:
            W = self.K(m)
            Xs = X + self.dt * (W + self.ad(v, X))
            s = m - self.dt * (self.ad_star(W, mu) + self.ad_star(v, m))
            Ws = self.K(s)
            if keep is not None:
                keep.append((m, W, s, Ws))
            X = 0.5 * X + 0.5 * (Xs + self.dt * (Ws + self.ad(vs, Xs)))
            m = 0.5 * m + 0.5 * (s - self.dt * (self.ad_star(Ws, ms) + self.ad_star(vs, s)))
        return X

    def hessvec(self, dv):
        X = self.tangent(dv)
        return 2.0 * dv + self.backward(2.0 / SIGMA2 * (self.G * X).sum(0) * self.G)

    def newton(self, dv):
        first, var = [], []
        self.backward(-2.0 / SIGMA2 * self.res * self.G, first)
        X = self.tangent(dv, var)
        s, c = -(self.G * X).sum(0), -2.0 / SIGMA2
        U = c * s * self.G + c * self.res * self.grad(s)
        w = torch.zeros_like(U)
        for (mu, v, ms, vs), (U1, w1, U2, w2), (m, W, sm, Ws) in zip(reversed(self.path), first, reversed(var)):
            Z = U + self.ad_star(w, ms) + self.ad_star(w1, sm)
            Us = U + self.dt * (self.ad_star(vs, U) + self.ad_star(Ws, U1))
            ws = w + self.dt * (self.K(Z) - self.ad(vs, w) - self.ad(Ws, w1))
            Z = Us + self.ad_star(ws, mu) + self.ad_star(w2, m)
            U = 0.5 * U + 0.5 * (Us + self.dt * (self.ad_star(v, Us) + self.ad_star(W, U2)))
            w = 0.5 * w + 0.5 * (ws + self.dt * (self.K(Z) - self.ad(v, ws) - self.ad(W, w2)))
        return 2.0 * dv + w

    def solve(self, iters, cg):
        v = torch.zeros((3,) + self.n, device=DEV, dtype=torch.float64)
        self.shoot(v)
        first, g0 = self.E, None
        for _ in range(iters):
            g = self.gradient(v)
            Lg = self.L(g)
            norm = math.sqrt(self.inner(Lg, g))
            g0 = norm if g0 is None else g0
            x, r, Lr = torch.zeros_like(g), -g, -Lg
            p, Lp, rr = r, Lr, self.inner(Lg, g)
            for _ in range(cg):
                H = self.hessvec(p)
                a = rr / self.inner(Lp, H)
                x, r = x + a * p, r - a * H
                Lr = self.L(r)
                new = self.inner(Lr, r)
                if math.sqrt(new) <= min(0.5, math.sqrt(norm / g0)) * norm:
                    break
                p, Lp, rr = r + new / rr * p, Lr + new / rr * Lp, new
            slope, E0, tau = self.inner(Lg, x), self.E, 1.0
            self.shoot(v + tau * x)
            while self.E > E0 + 1e-4 * tau * slope:
                tau *= 0.5
                self.shoot(v + tau * x)
            v = v + tau * x
        base = self.inner(self.I0 - self.I1, self.I0 - self.I1)
        mse = 100.0 * self.inner(self.res, self.res) / base
        return {"v0": v, "energy": [first, self.E], "mse_rel": mse}

    def pde(self, v, dv, stationary):
        nt, dt = self.nt, self.dt
        at = (lambda f, k: f) if stationary else (lambda f, k: f[k])
        div = lambda f: sum(self.d(f[e], e) for e in range(3))  # noqa: E731
        m, lines, feet = [self.I0], [], []
        for k in range(nt):
            x = self.foot(at(v, k), at(v, k + 1))
            feet.append(self.vox(x))
            m.append(self.at(m[k], feet[k]))
        for k in range(nt):
            a, b = at(v, k), at(v, k + 1)
            y = self.vox(0.5 * dt * (a + self.at(b, self.vox(dt * a))))
            lines.append((y, torch.exp(0.5 * dt * (div(a) + self.at(div(b), y)))))
        w = [dt * (0.5 if k in (0, nt) else 1.0) for k in range(nt + 1)]

        def back(lam, base):
            acc = torch.zeros_like(base)
            for k in range(nt, -1, -1):
                if k < nt:
                    lam = self.at(lam, lines[k][0]) * lines[k][1]
                if stationary:
                    acc += w[k] * lam * self.grad(m[k])
                else:
                    acc[k] = 2.0 * self.L(base[k]) + lam * self.grad(m[k])
            return acc + 2.0 * self.L(base) if stationary else acc

        r = m[nt] - self.I1
        steps = [0] if stationary else range(nt + 1)
        reg = sum((1.0 if stationary else w[k]) * self.inner(self.L(at(v, k)), at(v, k)) for k in steps)
        g = back(-2.0 / SIGMA2 * r, v)
        dm, s = torch.zeros_like(self.I0), -(self.grad(m[0]) * at(dv, 0)).sum(0)
        for k in range(nt):
            s2 = -(self.grad(m[k + 1]) * at(dv, k + 1)).sum(0)
            dm, s = self.at(dm, feet[k]) + 0.5 * dt * (self.at(s, feet[k]) + s2), s2
        return {"g": g, "energy": reg + self.inner(r, r) / SIGMA2, "hv": back(-2.0 / SIGMA2 * dm, dv)}


def exact(case, seed):
    a = {k: x.double() for k, x in _inputs(case, seed).items()}
    E, op = _Exact(case, a), case["op"]
    if op == "operator":
        return (E.L if case["L"] else E.K)(a["f"])
    if op == "solve":
        return E.solve(case["iters"], case["cg"])
    if op == "pde":
        return E.pde(a["v0"], a["dv"], case["stationary"])
    u, v = E.shoot(a["v0"])
    if op == "shoot":
        J = torch.stack([E.grad(u[c]) for c in range(3)])
        for c in range(3):
            J[c, c] += 1.0
        det = (J[0, 0] * (J[1, 1] * J[2, 2] - J[1, 2] * J[2, 1]) - J[0, 1] * (J[1, 0] * J[2, 2] - J[1, 2] * J[2, 0])
               + J[0, 2] * (J[1, 0] * J[2, 1] - J[1, 1] * J[2, 0]))
        return {"J1": E.J1, "u1": u, "v1": v, "energy": E.E, "det": det, "det_min": float(det.min()),
                "det_max": float(det.max())}
    if op == "gradient":
        return {"g": E.gradient(a["v0"]), "energy": E.E}
    if op == "hessvec":
        return E.hessvec(a["dv"])
    if op == "newton":
        return E.newton(a["dv"])
    return {"J1": E.J1, "grad": E.L(E.backward(-E.res * E.G))}
