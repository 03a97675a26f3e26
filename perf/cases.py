"""Workloads on which the solver's and the surrogate's speed is measured.

Two kinds of pass, each through the package's public entry points:

* "solver": a batch of instances advanced by a number of time steps, then read
  out the way the drivers do (coarse snapshots for the surrogate's data, the
  field itself, or the order parameter of every instance beside the field).
* "rollout" / "train": one step of the surrogate's rollout (network in place,
  projection, norms) and a few of its training steps.

A solver case is described by the instance counts per grid size (n64, n128,
...), the coefficient preset, the arithmetic, the scheme, the steps of a pass,
the graph length and the read-out.  Instances of one case share the grid
spacing of their preset's driver, with radii spread over that driver's range.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2304_03306_amd import fno as F
from paper_2304_03306_amd import ttsh as T
from paper_2304_03306_amd import workloads as W

SIZES = (64, 128, 256, 512, 1024, 2048, 4096, 8192)
PRECISION = {"fp32": T.TTSH_FP32, "fp64": T.TTSH_FP64, "state64": T.TTSH_FP32_STATE64}


def _solver(name, preset, steps, out, graph=50, tune=20, prec="fp32", scheme="ifeuler", **counts):
    c = {"name": name, "kind": "solver", "preset": preset, "prec": prec, "scheme": scheme, "steps": steps,
         "graph": graph, "tune": tune, "out": out}
    c.update(counts)
    return c


def listed():
    return [
        # the smallest workload: one circle on 64^2 in FP64; launches and latency are all it costs
        _solver("circle 64 fp64", "workload", 100, "field", n64=1, prec="fp64"),
        # one circle on 512^2 alone, the single-instance parity workload
        _solver("circle 512", "workload", 100, "native", n512=1),
        # the radius sweep's ramps between two looks at the fields
        _solver("radius sweep", "workload", 200, "coarse", n128=12, n256=16, n512=36),
        # collecting the surrogate's training data: a coarse snapshot of every instance each 20 steps
        _solver("collect snapshots", "workload", 20, "coarse", graph=20, n128=12, n256=16, n512=36),
        # dumbbell cavities on 1024^2, beyond what the caches hold
        _solver("dumbbells 1024", "dumbbell", 50, "native", n1024=16),
        # hysteresis ramps at the paper's coefficients: order parameter of every circle each 100 steps
        _solver("paper ramps 512", "paper", 100, "order", graph=100, n512=24),
        # the paper's circles at an intermediate resolution
        _solver("paper circles 2048", "paper", 20, "native", graph=20, tune=5, n2048=6),
        # the paper's production grid
        _solver("paper circle 8192", "paper", 10, "native", graph=10, tune=3, n8192=1),
        # Lyapunov runs: a base state and its perturbed copies in FP64
        _solver("copies 512 fp64", "paper", 50, "field", prec="fp64", n512=10),
        # the fourth-order scheme on part of the sweep
        _solver("etdrk4 sweep", "workload", 20, "native", scheme="etdrk4", graph=20, n128=4, n256=6, n512=12),
        # one surrogate step of all 64 instances of the sweep
        {"name": "rollout step", "kind": "rollout", "batch": 64, "size": 128, "modes": 16, "layers": 4, "cin": 3},
        # training steps at the drivers' batch size, then the parameters for a checkpoint
        {"name": "training", "kind": "train", "batch": 256, "size": 128, "modes": 16, "layers": 4, "cin": 3,
         "steps": 4},
    ]


def draw(rng):
    kind = rng.choice(["solver"] * 7 + ["rollout"] * 2 + ["train"])
    if kind == "solver":
        preset = rng.choice(["workload", "workload", "dumbbell", "paper", "paper"])
        prec = rng.choice(["fp32"] * 5 + ["fp64", "state64"])
        scheme = rng.choice(["ifeuler"] * 5 + ["etd1", "etdrk2", "etdrk4"])
        stages = {"etdrk2": 2, "etdrk4": 4}.get(scheme, 1)
        top = int(10 ** rng.uniform(3.6, 7.2))  # grid points of a step
        c = _solver("", preset, 0, "", prec=prec, scheme=scheme)
        del c["name"]
        points = 0
        mix = rng.random() < 0.35
        fits = [n for n in SIZES if n * n <= max(top, 4096) and n <= 4096 and (n < 4096 or prec == "fp32")]
        for n in (rng.sample(fits, min(len(fits), 3)) if mix else [rng.choice(fits[-4:])]):
            most = max(1, min(96, top // (n * n * (2 if mix else 1))))
            c["n%d" % n] = rng.randint(max(1, most // 3), most)
            points += c["n%d" % n] * n * n
        cost = max(20e-6, points / 6e10) * stages * (3 if prec == "fp64" else 1)
        c["steps"] = max(3, min(rng.randint(15, 130), int(0.012 / cost)))
        c["graph"] = rng.choice([20, 50, 100])
        c["tune"] = rng.choice([0, 5])
        count = sum(v for k, v in c.items() if k[0] == "n" and k[1:].isdigit())
        outs = ["field"] if prec == "fp64" else ["native", "coarse"] if count <= 48 else ["coarse"]
        c["out"] = rng.choice(outs + (["order"] if prec == "fp32" and count <= 48 else []))
        if c["out"] in ("native", "order", "field") and points > 2.0e7:
            c["out"] = "coarse"
        return c
    size, modes = rng.choice([(128, 16), (128, 16), (128, 16), (128, 32), (64, 16)])
    c = {"kind": kind, "size": size, "modes": modes, "layers": rng.choice([4, 4, 2]), "cin": rng.choice([3, 3, 4])}
    top = 256 if modes == 16 else 64
    c["batch"] = int(round(math.exp(rng.uniform(0.0, math.log(top)))))
    if kind == "train":
        c["steps"] = rng.randint(1, 4)
    return c


# ---- inputs ----------------------------------------------------------------------------

def _counts(case):
    return [(n, case["n%d" % n]) for n in SIZES if case.get("n%d" % n)]


def _instances(case):
    """(N, L, centres, radii) of every instance, sizes in increasing order."""
    out = []
    for N, count in _counts(case):
        for i in range(count):
            f = (i + 0.5) / count
            if case["preset"] == "paper":  # circles about the vortex-pair transition, box as the drivers'
                L = 40.96 if N >= 1024 else 20.48
                out.append((N, L, [(0.0, 0.0)], [5.0 + f]))
            elif case["preset"] == "dumbbell":  # two overlapping chambers, their distance varied
                L = 0.25 * N
                d = L * (40.0 + 40.0 * f) / 256.0
                R = L * 40.0 / 256.0
                out.append((N, L, [(-d / 2, 0.0), (d / 2, 0.0)], [R, R]))
            else:  # the sweep's circles: spacing up to 0.5, L = 3.2 R
                L = N * (0.25 + 0.25 * f)
                out.append((N, L, [(0.0, 0.0)], [L / 3.2]))
    return out


def _coefficients(case):
    p = W.paper_coefficients() if case["preset"] == "paper" else W.workload_coefficients()
    return dataclasses.replace(p, scheme=case["scheme"])


def _flow(N, L, gen):
    """A random field [2][N][N] of unit size whose modes lie where the linear
    operator feeds the flow (|k| up to 1.5), as a developed state has them."""
    mc = max(2, min(N // 8, int(1.5 * L / (2 * math.pi))))
    q = torch.randn(2, 2 * mc + 1, mc + 1, 2, generator=gen, device="cuda", dtype=torch.float64)
    h = torch.zeros(2, N, N // 2 + 1, device="cuda", dtype=torch.complex128)
    h[:, :mc + 1, :mc + 1] = torch.view_as_complex(q[:, :mc + 1].contiguous())
    h[:, N - mc:, :mc + 1] = torch.view_as_complex(q[:, mc + 1:].contiguous())
    v = torch.fft.irfft2(h, s=(N, N))
    return (v * (0.4 / v.std())).float().double()


def _outside(N, L, centers, radii):
    """1 where a node lies outside every disk, uint8 on the GPU."""
    c = (torch.arange(N, device="cuda", dtype=torch.float64) - N // 2) * (L / N)
    out = torch.ones(N, N, dtype=torch.bool, device="cuda")
    for (cx, cy), R in zip(centers, radii):
        out &= ((c[None, :] - cx) ** 2 + (c[:, None] - cy) ** 2).sqrt() >= R
    return out.to(torch.uint8)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _coarse_size(case):
    return min(128, max(n for n, _ in _counts(case)))


def _parameters(case, seed):
    """Flat float32 parameters of the network, drawn as its own initialisation draws them."""
    C, hid, m, cin = 32, 128, case["modes"], case["cin"]
    rng = np.random.default_rng(seed)

    def normal(*shape, s=1.0):
        return (rng.standard_normal(shape) * s).astype(np.float32)

    parts = {"Pw": normal(cin, C, s=cin ** -0.5), "Pb": normal(C, s=0.1)}
    for l in range(case["layers"]):
        parts["Rr%d" % l] = (rng.random((2 * m, m, C, C)) / (C * C)).astype(np.float32)
        parts["Ri%d" % l] = (rng.random((2 * m, m, C, C)) / (C * C)).astype(np.float32)
        parts["W%d" % l] = normal(C, C, s=C ** -0.5)
        parts["b%d" % l] = normal(C, s=0.1)
    parts.update(Q1w=normal(C, hid, s=C ** -0.5), Q1b=normal(hid, s=0.1), Q2w=normal(hid, 2, s=hid ** -0.5),
                 Q2b=normal(2, s=0.1))
    return parts


def _samples(case, seed, batch):
    """Coarse fields [batch][n][n][cin]: a flow inside a circle, the mask, and the spacing if asked for."""
    n, gen = case["size"], _generator(seed)
    x = torch.empty(batch, n, n, case["cin"], device="cuda")
    for i in range(batch):
        L = n * (0.25 + 0.25 * (i + 0.5) / batch)
        c = (torch.arange(n, device="cuda", dtype=torch.float64) - n // 2) * (L / n)
        K = 0.5 * (1 + torch.tanh(((c[None, :] ** 2 + c[:, None] ** 2).sqrt() - L / 3.2) / 0.5))
        x[i, :, :, :2] = (_flow(n, L, gen) * (1 - K)).permute(1, 2, 0)
        x[i, :, :, 2] = K
        if case["cin"] > 3:
            x[i, :, :, 3] = L / n
    return x


def prepare(case, seed):
    if case["kind"] == "solver":
        inst, gen = _instances(case), _generator(seed)
        s = T.Solver([i[0] for i in inst], [i[1] for i in inst], _coefficients(case), PRECISION[case["prec"]])
        s.option(T.TTSH_OPT_GRAPH_STEPS, case["graph"])
        for q, (N, L, centers, radii) in enumerate(inst):
            if case["preset"] == "paper":
                s.mask_from_binary(q, _outside(N, L, centers, radii))
            else:
                s.mask_tanh(q, centers, radii, 0.5)
            s.set_field(q, _flow(N, L, gen))
        if case["tune"]:
            s.tune(case["tune"])
        if case["out"] == "coarse":
            n = _coarse_size(case)
            out = torch.empty(len(inst), n, n, 2, device="cuda")
        elif case["out"] == "field":
            out = [torch.empty(k, 2, n, n, device="cuda", dtype=torch.float64) for n, k in _counts(case)]
        else:
            out = [torch.empty(k, n, n, 2, device="cuda") for n, k in _counts(case)]
        return {"case": case, "solver": s, "out": out}
    n, B = case["size"], case["batch"]
    net = F.FNO(width=32, modes=case["modes"], layers=case["layers"], cin=case["cin"], cout=2, hidden=128, H=n, W=n,
                max_batch=B, seed=seed)
    net.set_params(np.concatenate([p.ravel() for p in _parameters(case, seed).values()]))
    st = {"case": case, "net": net}
    if case["kind"] == "rollout":
        st["x0"] = _samples(case, seed, B)
        st["x"] = torch.empty_like(st["x0"])
        st["solver"] = T.Solver([n], [0.5 * n], W.workload_coefficients(), T.TTSH_FP32)
    else:
        st["data"] = [_samples(case, seed + 1 + k, B) for k in range(2)]
        # targets: the fields one small change on
        st["target"] = [(x[..., :2] * 0.9 + 0.1 * x[..., :2].roll(1, 2)).contiguous() for x in st["data"]]
        st["y"] = torch.empty_like(st["target"][0])
    return st


# ---- one pass ----------------------------------------------------------------------------

def run(state):
    case = state["case"]
    if case["kind"] == "solver":
        s, out = state["solver"], state["out"]
        s.step(case["steps"])
        if case["out"] == "coarse":
            for i in range(len(s.N)):
                s.field_coarse(i, out.shape[1], out[i], 2)
            return out
        i, psi = 0, []
        for o in out:
            for k in range(o.shape[0]):
                if case["out"] == "field":
                    T.ttsh_get_field(s.ctx, i, o[k])
                else:
                    if case["out"] == "order":
                        psi.append(s.order(i)[0])
                    s.field_coarse(i, o.shape[1], o[k], 2)
                i += 1
        return {"fields": out, "psi": torch.tensor(psi)} if psi else out
    net, B = state["net"], case["batch"]
    if case["kind"] == "rollout":
        x = state["x"]
        x.copy_(state["x0"])
        net.forward_ex(x, x, case["cin"], True, B)
        norms = state["solver"].project_coarse(case["size"], x, case["cin"], B, norms=True)
        return {"x": x, "norms": norms}
    losses = []
    for k in range(case["steps"]):
        net.forward_ex(state["data"][k % 2], state["y"], 2, True, B, train=True)
        losses.append(net.loss(state["y"], state["target"][k % 2]))
        net.backward(B)
        net.adam_step(1e-4)
    return {"loss": torch.tensor(losses), "params": net.params()}


# ---- what a pass cannot do without ---------------------------------------------------------

def work(case):
    if case["kind"] == "solver":
        wide = 8 if case["prec"] == "fp64" else 4
        state = 4 if case["prec"] == "fp32" else 8
        stages = {"etdrk2": 2, "etdrk4": 4}.get(case["scheme"], 1)
        rows = 5 + (1 if case["preset"] == "paper" else 0)  # real transforms of a right-hand side
        nbytes = flops = 0.0
        for N, k in _counts(case):
            modes = math.pi * (N // 4) ** 2 / 2
            step = 2 * 2 * 2 * state * modes + stages * wide * N * N  # the state in and out, the mask
            nbytes += k * (case["steps"] * step + (8 if case["prec"] != "fp64" else 16) * (
                min(N, _coarse_size(case)) if case["out"] == "coarse" else N) ** 2)
            # 2.5 N^2 log2 N^2 per full real transform, of which half the columns' part is pruned
            one = rows * 0.75 * 2.5 * N * N * 2 * math.log2(N) + 40 * N * N
            flops += k * case["steps"] * stages * one
        return {"bytes": nbytes, "flops": flops}
    P, m, C = case["batch"] * case["size"] ** 2, case["modes"], 32
    per_layer = 2.0 * P * C * (C + 2 * m + 2 * m) + 8.0 * case["batch"] * 2 * m * m * C * C
    net = case["layers"] * per_layer + 2.0 * P * (case["cin"] * C + C * 128 + 128 * 2)
    params = case["layers"] * 4 * m * m * C * C
    if case["kind"] == "rollout":
        return {"bytes": P * 4.0 * (case["cin"] + 2 + 4) + 2.0 * params, "flops": net + 40.0 * P}
    # a training step keeps and re-reads each layer's input and pre-activation in 16 bits
    acts = 2.0 * P * C * (2 * case["layers"] + 1)
    step = P * 4.0 * (case["cin"] + 4) + 2 * acts + 4.0 * 7 * params
    return {"bytes": case["steps"] * step + 4.0 * params, "flops": case["steps"] * 3 * net}


# ---- the same passes in 64 bits --------------------------------------------------------------

class _Grid:
    """One instance's time step on the full half-spectrum (unitary transforms) in FP64."""

    def __init__(self, N, L, p, K):
        dev, f8 = "cuda", torch.float64
        self.N, self.p, self.K = N, p, K
        mx = torch.arange(N // 2 + 1, device=dev, dtype=f8)[None, :]
        my = torch.fft.fftfreq(N, 1.0 / N, device=dev, dtype=f8)[:, None]
        dk = 2 * math.pi / L
        self.kx, self.ky = dk * mx, dk * my
        self.k2 = self.kx ** 2 + self.ky ** 2
        self.keep = (mx ** 2 + my ** 2) <= (N // 4) ** 2
        self.ik2 = torch.where(self.k2 > 0, 1.0 / self.k2.clamp_min(1e-300), torch.zeros_like(self.k2))
        self.z = (-p.alpha - p.gamma0 * self.k2 - p.gamma2 * self.k2 ** 2) * p.dt

    def fwd(self, a):
        return torch.fft.rfft2(a, norm="ortho")

    def inv(self, a):
        return torch.fft.irfft2(a, s=(self.N, self.N), norm="ortho")

    def project(self, h):
        """Cutoff and divergence-free part of [x, y]."""
        d = (self.kx * h[0] + self.ky * h[1]) * self.ik2
        return [(h[0] - self.kx * d) * self.keep, (h[1] - self.ky * d) * self.keep]

    def start(self, v):
        return self.project([self.fwd(v[0]), self.fwd(v[1])])

    def forcing(self, u):
        p = self.p
        vx, vy = self.inv(u[0]), self.inv(u[1])
        om = self.inv(1j * (self.kx * u[1] - self.ky * u[0]))
        s = p.beta * (vx * vx + vy * vy) + p.gamma_v * self.K
        r = [-s * vx, -s * vy]
        f = [self.fwd(r[0] + p.lambda0 * om * vy), self.fwd(r[1] - p.lambda0 * om * vx)]
        mean = [r[0].sum() / self.N, r[1].sum() / self.N]
        if p.gamma_w == 0.0:
            return f, mean
        g = self.fwd(-p.gamma_w * self.K * om) * self.ik2
        # the vorticity source as a velocity, folded into the forcing
        h = self.project(f)
        return [h[0] + 1j * self.ky * g, h[1] - 1j * self.kx * g], mean

    def stage(self, base, a, terms):
        """a base + sum of w f over terms (w, (f, mean)), with the rule for the mean flow."""
        out = self.project([a * base[c] + sum(w * self.p.dt * f[0][c] for w, f in terms) for c in range(2)])
        for c in range(2):
            out[c][0, 0] = a[0, 0] * base[c][0, 0] + sum(w[0, 0] * self.p.dt * f[1][c] for w, f in terms)
            col = out[c][:, 0].clone()
            out[c][:, 0] = 0.5 * (col + torch.roll(torch.flip(col, [0]), 1).conj())
        return out

    @staticmethod
    def phis(z):
        small = z.abs() < 0.5
        zs = torch.where(small, torch.ones_like(z), z)
        p = [torch.expm1(zs) / zs]
        p.append((p[0] - 1.0) / zs)
        p.append((p[1] - 0.5) / zs)
        out = []
        for k in range(3):
            ser = sum(z ** j / math.factorial(j + k + 1) for j in range(18))
            out.append(torch.where(small, ser, p[k]))
        return out

    def step(self, u):
        z, scheme = self.z, self.p.scheme
        if scheme in ("ifeuler", "etd1", "imex"):
            if scheme == "imex":
                a = b = 1.0 / (1.0 - z)
            else:
                a = torch.exp(z)
                b = a if scheme == "ifeuler" else self.phis(z)[0]
            return self.stage(u, a, [(b, self.forcing(u))])
        if scheme == "etdrk2":
            p1, p2, _ = self.phis(z)
            fu = self.forcing(u)
            a = self.stage(u, torch.exp(z), [(p1, fu)])
            return self.stage(a, torch.ones_like(z), [(p2, self.forcing(a)), (-p2, fu)])
        e, q = torch.exp(0.5 * z), 0.5 * self.phis(0.5 * z)[0]
        p1, p2, p3 = self.phis(z)
        fu = self.forcing(u)
        a = self.stage(u, e, [(q, fu)])
        fa = self.forcing(a)
        b = self.stage(u, e, [(q, fa)])
        fb = self.forcing(b)
        fc = self.forcing(self.stage(a, e, [(2 * q, fb), (-q, fu)]))
        w = 2.0 * (p2 - 2.0 * p3)
        return self.stage(u, torch.exp(z), [(p1 - 3.0 * p2 + 4.0 * p3, fu), (w, fa), (w, fb), (-p2 + 4.0 * p3, fc)])


def _exact_mask(case, N, L, centers, radii):
    if case["preset"] == "paper":  # low-passed binary field, squared
        b = torch.fft.fft2(_outside(N, L, centers, radii).double())
        m = torch.fft.fftfreq(N, 1.0 / N, device="cuda", dtype=torch.float64)
        b = torch.where(m[None, :] ** 2 + m[:, None] ** 2 > (N // 8) ** 2, torch.zeros_like(b), b)
        return torch.fft.ifft2(b).real ** 2
    c = (torch.arange(N, device="cuda", dtype=torch.float64) - N // 2) * (L / N)
    K = torch.ones(N, N, device="cuda", dtype=torch.float64)
    for (cx, cy), R in zip(centers, radii):
        K *= 0.5 * (1 + torch.tanh((((c[None, :] - cx) ** 2 + (c[:, None] - cy) ** 2).sqrt() - R) / 0.5))
    return K


def _resample(u, N, n):
    """Half-spectra on an N grid taken to an n grid by mode, inside both grids' radius."""
    if N == n:
        return u
    out = []
    M = min(N, n) // 4
    for h in u:
        o = torch.zeros(n, n // 2 + 1, device="cuda", dtype=torch.complex128)
        o[:M + 1, :M + 1] = h[:M + 1, :M + 1]
        o[n - M:, :M + 1] = h[N - M:, :M + 1]
        my = torch.fft.fftfreq(n, 1.0 / n, device="cuda", dtype=torch.float64)[:, None]
        mx = torch.arange(n // 2 + 1, device="cuda", dtype=torch.float64)[None, :]
        out.append(o * (mx ** 2 + my ** 2 <= M * M) * (n / N))
    return out


def _psi(v, L):
    """Vortex order parameter about the centre."""
    n = v[0].shape[-1]
    c = (torch.arange(n, device="cuda", dtype=torch.float64) - n // 2) * (L / n)
    x, y = c[None, :], c[:, None]
    r = (x * x + y * y).sqrt()
    num = torch.where(r > 0, ((x * v[1] - y * v[0]) / r.clamp_min(1e-300)).abs(), torch.zeros_like(r)).sum()
    return ((num / (v[0] ** 2 + v[1] ** 2).sqrt().sum() - 2 / math.pi) / (1 - 2 / math.pi)).item()


def _exact_solver(case, seed):
    cost = sum(k * n * n for n, k in _counts(case)) * case["steps"] * {"etdrk2": 2, "etdrk4": 4}.get(case["scheme"], 1)
    launches = sum(k for _, k in _counts(case)) * case["steps"]
    if cost > 4e9 or launches > 14000:
        return None
    p, gen = _coefficients(case), _generator(seed)
    fields, psi = {}, []
    for N, L, centers, radii in _instances(case):
        g = _Grid(N, L, p, _exact_mask(case, N, L, centers, radii))
        u = g.start(_flow(N, L, gen))
        for _ in range(case["steps"]):
            u = g.step(u)
        if case["out"] == "order":
            psi.append(_psi([g.inv(u[0]), g.inv(u[1])], L))
        n = _coarse_size(case) if case["out"] == "coarse" else N
        v = [torch.fft.irfft2(h, s=(n, n), norm="ortho") for h in _resample(u, N, n)]
        fields.setdefault(n, []).append(torch.stack(v, 0 if case["out"] == "field" else -1))
    out = [torch.stack(f) for f in fields.values()]
    if case["out"] == "coarse":
        return out[0]
    return {"fields": out, "psi": torch.tensor(psi, dtype=torch.float64)} if psi else out


def _network(case, p, x):
    """The network on [B][n][n][cin] in FP64."""
    m, n = case["modes"], case["size"]
    rows = torch.cat([torch.arange(m), torch.arange(n - m, n)]).cuda()
    h = x @ p["Pw"] + p["Pb"]
    for l in range(case["layers"]):
        f = torch.fft.rfft2(h, dim=(1, 2))[:, rows, :m]
        R = torch.complex(p["Rr%d" % l], p["Ri%d" % l])
        g = torch.matmul(f.permute(1, 2, 0, 3).contiguous(), R).permute(2, 0, 1, 3)
        full = torch.zeros(x.shape[0], n, m, 32, device="cuda", dtype=torch.complex128).index_copy(1, rows, g)
        s = torch.fft.irfft2(torch.nn.functional.pad(full, (0, 0, 0, n // 2 + 1 - m)), s=(n, n), dim=(1, 2))
        z = s + h @ p["W%d" % l] + p["b%d" % l]
        h = torch.nn.functional.gelu(z) if l + 1 < case["layers"] else z
    return torch.nn.functional.gelu(h @ p["Q1w"] + p["Q1b"]) @ p["Q2w"] + p["Q2b"]


def exact(case, seed):
    if case["kind"] == "solver":
        return _exact_solver(case, seed)
    p = {k: torch.from_numpy(v).cuda().double() for k, v in _parameters(case, seed).items()}
    n, B, chunk = case["size"], case["batch"], 16
    if case["kind"] == "rollout":
        x = _samples(case, seed, B).double()
        norms = torch.empty(B, 2, dtype=torch.float64)
        mx = torch.arange(n // 2 + 1, device="cuda", dtype=torch.float64)[None, :]
        my = torch.fft.fftfreq(n, 1.0 / n, device="cuda", dtype=torch.float64)[:, None]
        m2 = mx ** 2 + my ** 2
        keep, im2 = m2 <= (n // 4) ** 2, 1.0 / m2.clamp_min(1.0)
        weight = torch.where(mx == 0, 1.0, 2.0)
        with torch.no_grad():
            for b in range(0, B, chunk):
                v = x[b:b + chunk, :, :, :2] + _network(case, p, x[b:b + chunk])
                h = torch.fft.rfft2(v.permute(3, 0, 1, 2))
                d = (mx * h[0] + my * h[1]) * im2
                h = [(h[0] - mx * d) * keep, (h[1] - my * d) * keep]
                w = mx * h[1] - my * h[0]
                sums = [(weight * (h[0].abs() ** 2 + h[1].abs() ** 2)).sum((1, 2)), (weight * w.abs() ** 2).sum((1, 2))]
                norms[b:b + chunk] = torch.stack(sums, 1).cpu() / (n * n)
                x[b:b + chunk, :, :, :2] = torch.stack([torch.fft.irfft2(q, s=(n, n)) for q in h], -1)
        return {"x": x, "norms": norms}
    for q in p.values():
        q.requires_grad_(True)
    opt = torch.optim.Adam(list(p.values()), lr=1e-4, betas=(0.9, 0.999), eps=1e-8)
    losses = []
    for k in range(case["steps"]):
        x = _samples(case, seed + 1 + k % 2, B)
        t = (x[..., :2] * 0.9 + 0.1 * x[..., :2].roll(1, 2)).double()
        x = x.double()
        opt.zero_grad()
        total = 0.0
        for b in range(0, B, chunk):
            d = x[b:b + chunk, :, :, :2] + _network(case, p, x[b:b + chunk]) - t[b:b + chunk]
            part = (d.flatten(1).norm(dim=1) / t[b:b + chunk].flatten(1).norm(dim=1)).sum() / B
            part.backward()
            total += part.item()
        opt.step()
        losses.append(total)
    return {"loss": torch.tensor(losses, dtype=torch.float64),
            "params": torch.cat([q.detach().flatten() for q in p.values()])}
