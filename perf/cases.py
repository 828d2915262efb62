"""The work that a program using this framework has it do, as cases to time.

listed() names the cases, draw() gives more of the same ranges, prepare() makes
what a program holds before the call (start state, material, plan or server),
run() is one pass through the public entry points, work() the bytes and
operations a pass cannot do without, and exact() the same results from plain
torch and numpy in 64 bits.
"""
import math
import random

import numpy as np
import torch

from paper_2302_08843_amd import mm

MU0 = 4.0e-7 * math.pi
GAMMA = 2.21e5
SERVING_GRIDS = [(64, 64, 1), (128, 128, 2), (256, 64, 4), (256, 256, 8)]


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _case(kind, n, prec, material="uniform", **more):
    return dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], prec=prec, material=material, **more)


def listed():
    return [
        # the smallest call: one field of a single-layer film of the serving
        # stream (a program that evaluates fields one at a time pays launches)
        dict(_case("heff", (64, 64, 1), "fp32"), name="heff_64x64x1_fp32"),
        # a small ragged sample with everything per cell (vacuum holes, A, DMI)
        # in double, as in a validation or a device geometry
        dict(_case("rhs", (37, 21, 5), "fp64", "dmi"), name="rhs_37x21x5_fp64_dmi"),
        # a device of ordinary size on extents that are no powers of two
        dict(_case("rhs", (200, 120, 12), "fp32", "dmi"), name="rhs_200x120x12_fp32_dmi"),
        # the single-field throughput grid in both precisions
        dict(_case("heff", (256, 256, 16), "fp32"), name="heff_256x256x16_fp32"),
        dict(_case("heff", (256, 256, 16), "fp64"), name="heff_256x256x16_fp64"),
        # the largest grid, fields in both precisions
        dict(_case("heff", (512, 512, 64), "fp32"), name="heff_512x512x64_fp32"),
        dict(_case("heff", (512, 512, 64), "fp64"), name="heff_512x512x64_fp64"),
        # time integration with adaptive steps: the small LLG problem in double
        # (host decisions and launches count) and the largest grid in single
        dict(_case("step", (32, 32, 4), "fp64", steps=16), name="step_32x32x4_fp64"),
        dict(_case("step", (512, 512, 64), "fp32", steps=4), name="step_512x512x64_fp32"),
        # a multilayer stack of unequal heights
        dict(_case("layers", (512, 512, 8), "fp32"), name="layers_512x512x8_fp32"),
        # inverse design: forward with checkpoints and the gradient
        dict(_case("adjoint", (128, 128, 1), "fp32", "cells", steps=40, every=10),
             name="adjoint_128x128x1_fp32"),
        # a request server: time integrations of all four serving grids at once
        dict(kind="serve", prec="fp32", count=12, mix=0, ps=16, name="serve_12_fp32"),
    ]


def _extent(rng, lo, hi):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, v))


def _grid(rng, most, deepest=64):
    while True:
        n = (_extent(rng, 8, 512), _extent(rng, 8, 512),
             1 if rng.random() < 0.15 else _extent(rng, 1, deepest))
        if 256 <= n[0] * n[1] * n[2] <= most:
            return n


def draw(rng):
    kind = rng.choice(["heff", "heff", "heff", "rhs", "rhs", "rhs", "step", "step", "layers",
                       "adjoint", "serve"])
    prec = rng.choice(["fp32", "fp32", "fp64"])
    if kind == "heff":
        return _case("heff", _grid(rng, 1 << 23), prec, rng.choice(["uniform", "uniform", "cells"]))
    if kind == "rhs":
        return _case("rhs", _grid(rng, 1 << 22), prec, rng.choice(["uniform", "cells", "dmi"]))
    if kind == "step":
        return _case("step", _grid(rng, 1 << 21), prec, rng.choice(["uniform", "uniform", "cells"]),
                     steps=rng.randint(3, 16))
    if kind == "layers":
        n = _grid(rng, 1 << 20, 8)
        return _case("layers", (n[0], n[1], max(2, n[2])), prec)
    if kind == "adjoint":
        every = rng.choice([5, 8, 10])
        return _case("adjoint", _grid(rng, 1 << 15, 4), prec, "cells", steps=rng.randint(8, 40),
                     every=every)
    return dict(kind="serve", prec="fp32", count=rng.randint(2, 12), mix=rng.randrange(1 << 20),
                ps=rng.randint(4, 16))


# ---------------------------------------------------------------------------
# Inputs, from the seed alone
# ---------------------------------------------------------------------------
def _smooth(n, gen, dev, ell=6.0):
    """Low-passed Gaussian noise, normalised per cell (double)."""
    nx, ny, nz = n
    w = torch.randn((3, nz, ny, nx), generator=gen, device=dev, dtype=torch.float64)
    k2 = sum((torch.fft.fftfreq(q, device=dev, dtype=torch.float64) ** 2).reshape(s)
             for q, s in ((nz, (-1, 1, 1)), (ny, (1, -1, 1))))
    kx = torch.fft.rfftfreq(nx, device=dev, dtype=torch.float64)
    f = torch.exp(-2.0 * math.pi ** 2 * ell ** 2 * (k2 + kx ** 2))
    for c in range(3):
        w[c] = torch.fft.irfftn(torch.fft.rfftn(w[c]) * f, s=(nz, ny, nx))
        w[c] /= w[c].std()
    return w / w.norm(dim=0, keepdim=True)


def _inputs(case, seed, dev):
    """Everything a case is made of, as plain values and double tensors."""
    rng = random.Random(1000003 * seed + 17)
    gen = torch.Generator(device=dev)
    gen.manual_seed(rng.randrange(1 << 40))
    dt = torch.float32 if case["prec"] == "fp32" else torch.float64
    if case["kind"] == "serve":
        mix = random.Random(case["mix"])
        reqs = []
        for r in range(case["count"]):
            n = SERVING_GRIDS[r % 4 if case["mix"] == 0 else mix.randrange(4)]
            c = rng.uniform(3e-9, 5e-9)
            u = [rng.gauss(0, 1) for _ in range(3)]
            b = rng.uniform(0.0, 0.05) / MU0 / math.sqrt(sum(v * v for v in u))
            reqs.append(dict(n=n, d=(c, c, c), Ms=rng.uniform(4e5, 1.4e6),
                             A=rng.uniform(5e-12, 2e-11), Ku=rng.uniform(0.0, 5e4),
                             alpha=rng.uniform(0.1, 1.0), H=[b * v for v in u],
                             m0=_smooth(n, gen, dev).to(dt)))
        return dict(reqs=reqs, t_end=case["ps"] * 1e-12, rtol=1e-6)
    n = (case["nx"], case["ny"], case["nz"])
    nx, ny, nz = n
    shape = (nz, ny, nx)
    s = dict(n=n, d=(4e-9, 4e-9, 4e-9), Ms=rng.uniform(6e5, 1.2e6), A=rng.uniform(1e-11, 2e-11),
             Ku=rng.uniform(1e4, 5e4), alpha=rng.uniform(0.02, 0.5), dz=None, Ms_cell=None,
             A_cell=None, D=0.0, H=[rng.uniform(-2e4, 2e4) for _ in range(3)])
    s["m0"] = _smooth(n, gen, dev).to(dt)
    if case["kind"] == "layers":
        s["dz"] = [rng.uniform(0.8e-9, 4e-9) for _ in range(nz)]
    if case["material"] != "uniform":
        ms = s["Ms"] * (0.75 + 0.5 * torch.rand(shape, generator=gen, device=dev,
                                                dtype=torch.float64))
        if case["kind"] != "adjoint":  # vacuum holes; a trainable density has none
            ms = torch.where(torch.rand(shape, generator=gen, device=dev) < 0.1,
                             torch.zeros_like(ms), ms)
        s["Ms_cell"] = ms.to(dt)
    if case["material"] == "dmi":
        a = s["A"] * (0.6 + 0.8 * torch.rand(shape, generator=gen, device=dev,
                                             dtype=torch.float64))
        s["A_cell"] = a.to(dt)
        s["D"] = rng.uniform(1e-3, 3e-3)
    if case["kind"] == "step":
        s.update(rtol=1e-6, dt=3e-13, t_end=5e-13 * case["steps"])
    if case["kind"] == "adjoint":
        s["Ku"] = 0.0
        s.update(dt=1e-13, amp=[0.0, 0.02 / MU0, 0.0], freq=20e9,
                 strip=np.zeros(shape, np.uint8), region=np.zeros(shape, np.uint8))
        s["strip"][:, :, nx // 8:nx // 8 + 4] = 1
        s["region"][:, ny // 3:2 * ny // 3 + 1, 3 * nx // 4:7 * nx // 8 + 1] = 1
    return s


def prepare(case, seed):
    s = _inputs(case, seed, torch.device("cuda"))
    s["case"] = case
    if case["kind"] == "serve":
        s["server"] = mm.Server(budget=8 << 30, prec=case["prec"])
        return s
    plan = mm.Plan(s["n"], s["d"], s["Ms"], A=s["A"], Ku=s["Ku"], alpha=s["alpha"],
                   prec=case["prec"], layers=s["dz"])
    if s["Ms_cell"] is not None:
        plan.set_ms(s["Ms_cell"])
    if s["A_cell"] is not None:
        plan.set_exchange(s["A_cell"])
    if s["D"]:
        plan.set_dmi(s["D"], mm.MM_DMI_INTERFACE)
    if case["kind"] == "adjoint":
        plan.set_drive(s["amp"], s["freq"], s["strip"])
        s["region_dev"] = torch.from_numpy(s["region"]).cuda()
    s["plan"] = plan
    return s


def run(state):
    s, case = state, state["case"]
    kind = case["kind"]
    if kind == "serve":
        srv = s["server"]
        out = [q["m0"].clone() for q in s["reqs"]]
        for i, q in enumerate(s["reqs"]):
            srv.submit(out[i], q["n"], q["d"], q["Ms"], q["A"], Ku=q["Ku"], alpha=q["alpha"],
                       h_ext=q["H"], kind=mm.MM_SERVE_INTEGRATE, rtol=s["rtol"],
                       t_end=s["t_end"], tag=i)
        left = len(out)
        while left:
            for done in srv.poll():
                if done["status"] != mm.MM_OK:
                    raise RuntimeError("request %d: status %d" % (done["tag"], done["status"]))
                left -= 1
        return out
    plan = s["plan"]
    if kind in ("heff", "layers"):
        return plan.heff(s["m0"], s["H"], mm.MM_ALL)
    if kind == "rhs":
        return plan.llg_rhs(s["m0"], s["H"], mm.MM_ALL)
    m = s["m0"].clone()
    if kind == "step":
        plan.llg_step(m, s["H"], mm.MM_ALL, t=0.0, dt=s["dt"], rtol=s["rtol"], t_end=s["t_end"])
        return m
    loss, ck = plan.rk4(m, s["dt"], case["steps"], s["region_dev"], s["H"], mm.MM_ALL,
                        ckpt_every=case["every"])
    _, gms, gm0 = plan.rk4_adjoint(ck, s["dt"], case["steps"], s["region_dev"], s["H"], mm.MM_ALL,
                                   ckpt_every=case["every"])
    return dict(m=m, grad_ms=gms, grad_m0=gm0, loss=torch.tensor(loss, dtype=plan.dtype))


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _pad(n):
    return 1 if n == 1 else 1 << (2 * n - 2).bit_length()


def _field_work(n, size, layers=False, per_cell=0):
    """One field evaluation: the state in, the field out, the per-cell
    constants and the demag kernel's spectrum (real, one octant) once."""
    cells = n[0] * n[1] * n[2]
    P = [_pad(q) for q in n]
    if layers:
        P[2] = n[2]
    pts = P[0] * P[1] * P[2]
    lines = (P[0] // 2 + 1) * (P[1] // 2 + 1)
    kernel = 6 * lines * (n[2] * (n[2] + 1) // 2 if layers else P[2] // 2 + 1)
    byts = size * (6 * cells + per_cell * cells + kernel)
    lengths = P[:2] if layers else P
    flops = 6 * 2.5 * pts * math.log2(max(2, np.prod(lengths))) + 60 * cells
    flops += 15.0 * pts * (n[2] if layers else 1)
    return byts, flops


def work(case):
    size = 4 if case["prec"] == "fp32" else 8
    if case["kind"] == "serve":
        mix = random.Random(case["mix"])
        tot = [0.0, 0.0]
        for r in range(case["count"]):
            n = SERVING_GRIDS[r % 4 if case["mix"] == 0 else mix.randrange(4)]
            b, f = _field_work(n, size)
            # about two steps of six evaluations per picosecond
            tot[0] += 12 * case["ps"] * b
            tot[1] += 12 * case["ps"] * f
        return dict(bytes=tot[0], flops=tot[1])
    n = (case["nx"], case["ny"], case["nz"])
    cells = {"uniform": 0, "cells": 1, "dmi": 2}[case["material"]]
    b, f = _field_work(n, size, case["kind"] == "layers", cells)
    evals = 1
    if case["kind"] == "step":
        evals = 6 * case["steps"]
    if case["kind"] == "adjoint":  # forward, recomputed forward, transposed fields
        evals = 12 * case["steps"]
    return dict(bytes=float(evals * b), flops=float(evals * f))


# ---------------------------------------------------------------------------
# The same in 64 bits, from the formulas
# ---------------------------------------------------------------------------
def _newell(x, y, z, diag):
    """Newell's f (diagonal entries) or g (off-diagonal), in long double."""
    r = np.sqrt(x * x + y * y + z * z)

    def asinh(a, p, q):
        h = np.sqrt(p * p + q * q)
        return np.where(h > 0, np.arcsinh(a / np.where(h > 0, h, 1)), 0)

    def atan(num, den):
        return np.where(den != 0, np.arctan(num / np.where(den != 0, den, 1)), 0)

    if diag:
        x, y, z = abs(x), abs(y), abs(z)
        return (y / 2 * (z * z - x * x) * asinh(y, x, z) + z / 2 * (y * y - x * x) * asinh(z, x, y)
                - x * y * z * atan(y * z, x * r) + (2 * x * x - y * y - z * z) * r / 6)
    return (x * y * z * asinh(z, x, y) + y / 6 * (3 * z * z - y * y) * asinh(x, y, z)
            + x / 6 * (3 * z * z - x * x) * asinh(y, x, z) - z ** 3 / 6 * atan(x * y, z * r)
            - z * y * y / 2 * atan(x * z, y * r) - z * x * x / 2 * atan(y * z, x * r)
            - x * y * r / 3)


_PAIRS = [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)]


def _entry(comp, x, y, z):
    a, b = _PAIRS[comp]
    v = (x, y, z)
    if a == b:
        o = [q for q in range(3) if q != a]
        return _newell(v[a], v[o[0]], v[o[1]], True)
    return _newell(v[a], v[b], v[3 - a - b], False)


def _near(comp, n, d, p):
    """-N of uniform cells for offsets 0..p along each axis (double)."""
    u = d[0]
    ext = [min(q - 1, p) + 1 for q in n]
    ax = [np.arange(-1, e + 1, dtype=np.longdouble) * np.longdouble(h / u) for e, h in zip(ext, d)]
    F = _entry(comp, ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None])
    F = np.broadcast_to(F, tuple(len(a) for a in ax[::-1]))
    for k in range(3):
        F = np.moveaxis(F, k, 0)
        F = np.moveaxis(2 * F[1:-1] - F[:-2] - F[2:], 0, k)
    vol = np.longdouble(d[0] / u) * np.longdouble(d[1] / u) * np.longdouble(d[2] / u)
    return (-F / (4 * np.longdouble(np.pi) * vol)).astype(np.float64)


def _near_layer(comp, n, d, bottom, ht, hs, p):
    """-N between a target of height ht and a source of height hs whose bottom
    sits `bottom` above the target's."""
    u = d[0]
    ext = [min(q - 1, p) + 1 for q in n[:2]]
    ax = [np.arange(-1, e + 1, dtype=np.longdouble) * np.longdouble(h / u)
          for e, h in zip(ext, d[:2])]
    tot = 0
    for z, sg in ((bottom + hs, -1), (bottom + hs - ht, 1), (bottom, 1), (bottom - ht, -1)):
        zz = np.full((1, 1), np.longdouble(z) / np.longdouble(u))
        tot = tot + sg * _entry(comp, ax[0][None, :], ax[1][:, None], zz)
    for k in range(2):
        tot = np.moveaxis(tot, k, 0)
        tot = np.moveaxis(2 * tot[1:-1] - tot[:-2] - tot[2:], 0, k)
    vol = np.longdouble(d[1] / u) * np.longdouble(ht / u)
    return (-tot / (4 * np.longdouble(np.pi) * vol)).astype(np.float64)


def _offsets(n, P, dev):
    o = torch.arange(P, device=dev)
    return torch.where(o < n, o, torch.where(o > P - n, o - P, torch.full_like(o, 1 << 20)))


def _dipole(comp, r, vol):
    a, b = _PAIRS[comp]
    r2 = r[0] ** 2 + r[1] ** 2 + r[2] ** 2
    r2 = torch.where(r2 == 0, torch.ones_like(r2), r2)
    v = 3.0 * r[a] * r[b] / r2
    if a == b:
        v = v - 1.0
    return vol * v / (4.0 * math.pi * r2 * torch.sqrt(r2))


def _sign(comp, I, J, K):
    a, b = _PAIRS[comp]
    if a == b:
        return 1.0
    o = (I, J, K)
    return (1.0 - 2.0 * (o[a] < 0).double()) * (1.0 - 2.0 * (o[b] < 0).double())


class _Field:
    """The effective field and right-hand side in double torch."""

    def __init__(self, s, dev, p=20):
        self.s, self.dev, n, d = s, dev, s["n"], s["d"]
        self.P = [_pad(q) for q in n]
        self.dz = s.get("dz")
        X, Y, Z = (_offsets(n[a], self.P[a], dev) for a in range(3))
        big = 1 << 19
        if self.dz is None:
            I, J, K = X[None, None, :], Y[None, :, None], Z[:, None, None]
            ok = (I.abs() < big) & (J.abs() < big) & (K.abs() < big)
            near = ok & (I.abs() <= p) & (J.abs() <= p) & (K.abs() <= p)
            at = torch.nonzero(near)
            aI, aJ, aK = X[at[:, 2]].abs(), Y[at[:, 1]].abs(), Z[at[:, 0]].abs()
            r = [I.double() * d[0], J.double() * d[1], K.double() * d[2]]
            self.K = []
            for c in range(6):
                v = torch.where(ok, _dipole(c, r, d[0] * d[1] * d[2]), 0.0)
                t = torch.from_numpy(_near(c, n, d, p)).to(dev)
                sg = _sign(c, X[at[:, 2]], Y[at[:, 1]], Z[at[:, 0]])
                v[at[:, 0], at[:, 1], at[:, 2]] = sg * t[aK, aJ, aI]
                self.K.append(torch.fft.rfftn(v))
                del v
        else:
            zb = np.concatenate([[0.0], np.cumsum(self.dz)])
            I, J = X[None, :], Y[:, None]
            ok = (I.abs() < big) & (J.abs() < big)
            near = ok & (I.abs() <= p) & (J.abs() <= p)
            at = torch.nonzero(near)
            Io, Jo = X[at[:, 1]], Y[at[:, 0]]
            nz = n[2]
            self.K = [[[None] * nz for _ in range(nz)] for _ in range(6)]
            for c in range(6):
                for t in range(nz):
                    for q in range(nz):
                        # the field point is the target: its offset from the source
                        dzc = 0.5 * (zb[t] + zb[t + 1]) - 0.5 * (zb[q] + zb[q + 1])
                        r = [I.double() * d[0], J.double() * d[1],
                             torch.full((1, 1), dzc, dtype=torch.float64, device=dev)]
                        v = torch.where(ok, _dipole(c, r, d[0] * d[1] * self.dz[q]), 0.0)
                        w = _near_layer(c, n, d, zb[q] - zb[t], self.dz[t], self.dz[q], p)
                        w = torch.from_numpy(w).to(dev)
                        a, b = _PAIRS[c]
                        # offsets enter as source minus target along z and
                        # target minus source laterally
                        sg = 1.0
                        if a != b:
                            sx, sy = 1.0 - 2.0 * (Io < 0).double(), 1.0 - 2.0 * (Jo < 0).double()
                            sg = {3: sx * sy, 4: -sx, 5: -sy}[c]
                        v[at[:, 0], at[:, 1]] = sg * w[Jo.abs(), Io.abs()]
                        self.K[c][t][q] = torch.fft.rfftn(v)
        self.ms = (torch.full((n[2], n[1], n[0]), s["Ms"], dtype=torch.float64, device=dev)
                   if s.get("Ms_cell") is None else s["Ms_cell"].double())
        self.mag = self.ms > 0
        self.inv = torch.where(self.mag, 1.0 / torch.where(self.mag, self.ms, 1.0), 0.0)
        self.A = s.get("A_cell")
        self.A = None if self.A is None else self.A.double()
        self.H = torch.tensor(s["H"], dtype=torch.float64, device=dev).reshape(3, 1, 1, 1)
        self.drive = None
        if "strip" in s:
            self.drive = torch.from_numpy(s["strip"]).to(dev).double() * torch.tensor(
                s["amp"], dtype=torch.float64, device=dev).reshape(3, 1, 1, 1)

    def demag(self, m, ms):
        nx, ny, nz = self.s["n"]
        Px, Py, Pz = self.P
        M = ms * m
        order = ((0, 3, 4), (3, 1, 5), (4, 5, 2))
        if self.dz is None:
            F = [torch.fft.rfftn(M[c], s=(Pz, Py, Px)) for c in range(3)]
            out = []
            for a in range(3):
                G = sum(self.K[order[a][b]] * F[b] for b in range(3))
                out.append(torch.fft.irfftn(G, s=(Pz, Py, Px))[:nz, :ny, :nx])
            return torch.stack(out)
        F = [[torch.fft.rfftn(M[c, k], s=(Py, Px)) for k in range(nz)] for c in range(3)]
        out = torch.empty_like(M)
        for a in range(3):
            for t in range(nz):
                G = sum(self.K[order[a][b]][t][q] * F[b][q] for b in range(3) for q in range(nz))
                out[a, t] = torch.fft.irfftn(G, s=(Py, Px))[:ny, :nx]
        return out

    def stencil(self, m, inv):
        s, n = self.s, self.s["n"]
        ex, dm = torch.zeros_like(m), torch.zeros_like(m)
        edmi = ((0, 1.0, 0), (-1.0, 0, 0), None)  # interface DMI vectors of x, y, z
        for a in range(3):
            axis = 3 - a
            if n[a] == 1:
                continue
            for sgn in (-1, 1):
                lo = [slice(None)] * 4
                hi = [slice(None)] * 4
                lo[axis], hi[axis] = slice(0, n[a] - 1), slice(1, n[a])
                me, nb = (lo, hi) if sgn > 0 else (hi, lo)
                me, nb = tuple(me), tuple(nb)
                w = self.mag[nb[1:]].double()
                if self.dz is not None and a == 2:
                    h = torch.tensor(self.dz, dtype=torch.float64, device=self.dev)
                    w = w * (2.0 / (h[me[1]] * (h[me[1]] + h[nb[1]]))).reshape(-1, 1, 1)
                else:
                    w = w / s["d"][a] ** 2
                if self.A is None:
                    w = w * s["A"]
                else:
                    Ai, Aj = self.A[me[1:]], self.A[nb[1:]]
                    w = w * (2.0 * Ai * Aj / (Ai + Aj))
                ex[me] = ex[me] + w * (m[nb] - m[me])
                if s["D"] and edmi[a] is not None:
                    e = torch.tensor(edmi[a], dtype=torch.float64, device=self.dev)
                    e = (e * sgn * s["D"] / (2.0 * s["d"][a])).reshape(3, 1, 1, 1)
                    dm[me] = dm[me] + self.mag[nb[1:]].double() * torch.cross(
                        e.expand_as(m[nb]), m[nb], dim=0)
        return 2.0 / MU0 * inv * (ex + dm)

    def heff(self, m, t=0.0, ms=None):
        inv = self.inv if ms is None else 1.0 / ms
        h = self.demag(m, self.ms if ms is None else ms) + self.stencil(m, inv)
        an = torch.zeros_like(h)
        an[2] = 2.0 * self.s["Ku"] / MU0 * inv * m[2]
        h = h + an + self.H
        if self.drive is not None:
            h = h + self.drive * math.sin(2.0 * math.pi * self.s["freq"] * t)
        return torch.where(self.mag, h, 0.0)

    def rhs(self, m, t=0.0, ms=None):
        h, al = self.heff(m, t, ms), self.s["alpha"]
        p = torch.cross(m, h, dim=0)
        f = -GAMMA / (1.0 + al * al) * (p + al * torch.cross(m, p, dim=0))
        return torch.where(self.mag, f, 0.0)


_DPA = ((), (1 / 5,), (3 / 40, 9 / 40), (44 / 45, -56 / 15, 32 / 9),
        (19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729),
        (9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656),
        (35 / 384, 0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84))
_DPE = (71 / 57600, 0, -71 / 16695, 71 / 1920, -17253 / 339200, 22 / 525, -1 / 40)


def _integrate(f, y, dt, t_end, tol):
    """Adaptive Dormand-Prince 5(4) to t_end at a tolerance well below the
    case's own."""
    t, k0 = 0.0, f.rhs(y)
    while t < t_end * (1 - 1e-14):
        h = min(dt, t_end - t)
        k = [k0]
        for row in _DPA[1:]:
            y1 = y + sum(h * c * v for c, v in zip(row, k) if c)
            k.append(f.rhs(y1))
        e = sum(h * c * v for c, v in zip(_DPE, k) if c)
        err = float(((e / (tol + tol * torch.maximum(y.abs(), y1.abs()))) ** 2).mean().sqrt())
        if err <= 1.0:
            t, y, k0 = t + h, y1, k[6]
        dt = h * min(5.0, max(0.2, 0.9 * (err + 1e-30) ** -0.2))
    return y


def exact(case, seed, device=None):
    dev = torch.device(device or "cuda")
    s = _inputs(case, seed, dev)
    if case["kind"] == "serve":
        out = []
        for q in s["reqs"]:
            q = dict(q, D=0.0)
            out.append(_integrate(_Field(q, dev), q["m0"].double(), 1e-13, s["t_end"], 1e-8))
        return out
    f, m = _Field(s, dev), s["m0"].double()
    if case["kind"] in ("heff", "layers"):
        return f.heff(m)
    if case["kind"] == "rhs":
        return f.rhs(m)
    if case["kind"] == "step":
        return _integrate(f, m, 1e-13, s["t_end"], 1e-8)
    # classical Runge-Kutta with the region loss, differentiated by autograd
    ms = f.ms.clone().requires_grad_(True)
    m0 = m.clone().requires_grad_(True)
    region, y, dt, loss = torch.from_numpy(s["region"]).to(dev).bool(), m0, s["dt"], 0.0
    for i in range(case["steps"]):
        t = i * dt
        k1 = f.rhs(y, t, ms)
        k2 = f.rhs(y + dt / 2 * k1, t + dt / 2, ms)
        k3 = f.rhs(y + dt / 2 * k2, t + dt / 2, ms)
        k4 = f.rhs(y + dt * k3, t + dt, ms)
        y = y + dt / 6 * (k1 + 2 * k2 + 2 * k3 + k4)
        loss = loss + y[2][region].mean() / case["steps"]
    gms, gm0 = torch.autograd.grad(loss, (ms, m0))
    return dict(m=y.detach(), grad_ms=gms, grad_m0=gm0, loss=loss.detach())
