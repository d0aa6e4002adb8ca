"""What a user of this library has it do, as timed cases: stepping the solver and reading
the fields back, stepping an ensemble, the surrogate's forward pass, its gradients, and
single convolution layers.

A case is a dict of plain values; `prepare` makes the inputs and the handles a program
keeps, `run` is one pass through the public entry points, `exact` the same result in
float64 without the library, `work` the bytes and operations a pass cannot do without.
"""
import math
import random

import numpy as np
import torch

import pfinputs
from paper_1812_00118_amd import Sim
from paper_1812_00118_amd.surrogate import (HEAD, LAYERS, Surrogate, conv_fwd, conv_wgrad,
                                            init_params)

SAME, UP, POOL = 0, 1, 2


def listed():
    return [
        # The smallest domain in use: the paper's static droplet, stepped between two looks
        # at the fields.  Launches and latency count, not bytes.
        dict(name="static_droplet_64x64", what="step", physics="droplet", nx=64, ny=64, nz=1,
             storage="fp32", steps=16),
        # The paper's two-dimensional workload with walls and gravity.
        dict(name="rayleigh_taylor_256x1024", what="step", physics="rt", nx=256, ny=1024, nz=1,
             storage="fp32", steps=16),
        # The surrogate's data: an ensemble of small domains of different densities, stepped
        # together over the lead-in and read out.
        dict(name="drops_32x256x256", what="ensemble", domains=32, n=256, storage="fp32",
             steps=64),
        # The three-dimensional workload of the benchmark in each storage a program may pick.
        dict(name="rising_bubble_128_fp32", what="step", physics="bubble", nx=128, ny=128,
             nz=128, storage="fp32", steps=16),
        dict(name="rising_bubble_128_fp16s", what="step", physics="bubble", nx=128, ny=128,
             nz=128, storage="fp16s", steps=16),
        dict(name="rising_bubble_128_inplace", what="step", physics="bubble", nx=128, ny=128,
             nz=128, storage="fp32_inplace", steps=16),
        # The large three-dimensional workload.
        dict(name="droplet_impact_256x256x128", what="step", physics="impact", nx=256, ny=256,
             nz=128, storage="fp32", steps=16),
        # The paper's dam-break box: ragged in every axis, walls all round, an open top.
        dict(name="dam_break_537x50x198_fp16s", what="step", physics="dam", nx=537, ny=50,
             nz=198, storage="fp16s", steps=8),
        # One prediction for one domain (latency), and for a whole ensemble (throughput).
        dict(name="forward_1x256x256", what="forward", batch=1, H=256, W=256),
        dict(name="forward_32x256x256", what="forward", batch=32, H=256, W=256),
        # Gradients of one training batch of the size the training schedule uses.
        dict(name="gradients_16x256x256", what="gradients", batch=16, H=256, W=256),
        # One layer as a program that assembles its own network calls it: forward with the
        # pre-activation, and the weight gradient.
        dict(name="layer_64to64_16x128x128", what="layer", batch=16, H=128, W=128, Cin=64,
             Cout=64, mode=SAME),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: every kind of call, odd sizes among them."""
    what = rng.choice(["step2", "step2", "ensemble", "step3", "step3", "forward", "gradients",
                       "layer"])
    if what == "step2":
        physics = rng.choice(["droplet", "rt"])
        nx, ny = (_log(rng, 48, 700), _log(rng, 48, 700)) if physics == "droplet" else \
                 (_log(rng, 128, 512), _log(rng, 160, 1400))
        return dict(what="step", physics=physics, nx=nx, ny=ny, nz=1,
                    storage=rng.choice(["fp32", "fp32", "fp16s", "fp32_inplace"]),
                    steps=_log(rng, 1, 32))
    if what == "ensemble":
        return dict(what="ensemble", domains=_log(rng, 2, 32), n=_log(rng, 128, 256),
                    storage=rng.choice(["fp32", "fp32", "fp16s"]), steps=_log(rng, 4, 64))
    if what == "step3":
        physics = rng.choice(["bubble", "impact", "dam"])
        nx, ny, nz = (_log(rng, 48, 256) for _ in range(3))
        while nx * ny * nz > 256 * 256 * 128:
            nx, ny, nz = (max(48, int(v * 0.8)) for v in (nx, ny, nz))
        storage = rng.choice(["fp32", "fp32", "fp16s", "fp32_inplace"])
        if physics == "dam" and storage == "fp32_inplace":
            storage = "fp32"                     # in-place storage has no open faces
        return dict(what="step", physics=physics, nx=nx, ny=ny, nz=nz, storage=storage,
                    steps=_log(rng, 1, 16))
    if what == "layer":
        name, cin, cout = rng.choice(LAYERS[1:])
        mode = UP if name[0] == "u" else POOL if name in ("e1a", "e2a", "b3a") else SAME
        H, W = (2 * _log(rng, 8, 80) for _ in range(2))
        return dict(what="layer", batch=_log(rng, 1, 16), H=H, W=W, Cin=cin, Cout=cout,
                    mode=mode)
    H, W = (8 * _log(rng, 4, 32) for _ in range(2))
    return dict(what=what, batch=_log(rng, 1, 32 if what == "forward" else 16), H=H, W=W)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _config(case):
    """Parameters of a case's workload at the case's sizes."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    p = case["physics"]
    if p == "droplet":
        cfg = pfinputs.static_droplet(64, R=min(nx, ny) / 4.0)
    elif p == "rt":
        cfg = pfinputs.rayleigh_taylor(nx, ny)
    elif p == "bubble":
        cfg = pfinputs.rising_bubble(128, R=max(5.0, min(nx, ny, nz) / 8.0))
    elif p == "impact":
        cfg = pfinputs.droplet_impact(nx, ny, nz, R=min(nx, ny, nz) / 4.0, film=nz / 8.0)
    else:
        cfg = pfinputs.dam_break(nx, ny, nz, H=nz * 0.5, L=nx * 0.37)
    cfg["shape"] = (nx, ny, nz)
    return cfg


def _hydrostatic(cfg, phi):
    """dP/ds = rho g along the gravity axis, zero mean."""
    g = max(cfg["g"], key=abs)
    if g == 0.0:
        return torch.zeros_like(phi)
    dim = 2 - list(cfg["g"]).index(g)
    f = (cfg["rho_L"] + phi * (cfg["rho_H"] - cfg["rho_L"])) * g
    P = torch.cumsum(f, dim) - 0.5 * f - 0.5 * f.narrow(dim, 0, 1)
    return P - P.mean()


def _fields(cfg, seed):
    """phi, u, P (float32) of a workload: its own shape, placed and sized a little
    differently for each seed, in a slight swirl."""
    rng = random.Random(seed)
    dev = _device()
    nx, ny, nz = cfg["shape"]
    x = torch.arange(nx, dtype=torch.float64, device=dev).view(1, 1, nx)
    y = torch.arange(ny, dtype=torch.float64, device=dev).view(1, ny, 1)
    z = torch.arange(nz, dtype=torch.float64, device=dev).view(nz, 1, 1)
    W = cfg["W"]
    off = [rng.uniform(-2.0, 2.0) for _ in range(3)]
    size = rng.uniform(0.95, 1.05)

    def ball(cz, R):
        r2 = (x - (nx - 1) / 2.0 - off[0]) ** 2 + (y - (ny - 1) / 2.0 - off[1]) ** 2
        if nz > 1:
            r2 = r2 + (z - cz) ** 2
        return 0.5 - 0.5 * torch.tanh(2.0 * (torch.sqrt(r2) - R * size) / W)

    u = torch.zeros((3, nz, ny, nx), dtype=torch.float64, device=dev)
    name = cfg["name"]
    if name == "static_droplet":
        phi = ball(0.0, cfg["R"])
    elif name == "rising_bubble":
        phi = 1.0 - ball(nz / 4.0 + off[2], cfg["R"])
    elif name == "rayleigh_taylor":
        y0 = (ny - 1) / 2.0 + size * min(cfg["amp"], ny / 4.0) * torch.cos(
            2.0 * math.pi * (x + off[0]) / nx)
        phi = 0.5 + 0.5 * torch.tanh(2.0 * (y - y0) / W)
    elif name == "droplet_impact":
        drop = ball(cfg["film"] + W + cfg["R"] * size, cfg["R"])
        film = 0.5 - 0.5 * torch.tanh(2.0 * (z - (cfg["film"] - 0.5)) / W)
        phi = torch.maximum(film.expand_as(drop), drop)
        u[2] = -cfg["U"] * drop
    else:
        dx, dz = x - (cfg["L"] * size - 0.5), z - (cfg["H"] - 0.5 + off[2])
        out = torch.sqrt(dx.clamp(min=0.0) ** 2 + dz.clamp(min=0.0) ** 2)
        d = torch.where((dx > 0) | (dz > 0), out, torch.maximum(dx, dz)).expand(nz, ny, nx)
        phi = 0.5 - 0.5 * torch.tanh(2.0 * d / W)
    phi = phi.expand(nz, ny, nx).contiguous()
    P = _hydrostatic(cfg, phi)
    if name == "dam_break":
        P = P - P[-1:]                           # 0 in the open top layer
    amp, ph = 1e-3, rng.uniform(0.0, 2.0 * math.pi)
    u[0] += amp * torch.sin(2.0 * math.pi * y / ny + ph)
    u[1] += amp * torch.sin(2.0 * math.pi * x / nx + ph)
    return phi.float(), u.float(), P.float()


def _drops(n, seed):
    """One domain of the surrogate family, periodic, its drops moving."""
    cfg = pfinputs.drops(seed, n)
    dev = _device()
    x = torch.arange(n, dtype=torch.float64, device=dev).view(1, 1, n)
    y = torch.arange(n, dtype=torch.float64, device=dev).view(1, n, 1)
    phi = torch.zeros((1, n, n), dtype=torch.float64, device=dev)
    u = torch.zeros((3, 1, n, n), dtype=torch.float64, device=dev)
    for cx, cy, R, vx, vy in cfg["drops"]:
        dx, dy = (x - cx).abs(), (y - cy).abs()
        dx, dy = torch.minimum(dx, n - dx), torch.minimum(dy, n - dy)
        p = 0.5 - 0.5 * torch.tanh(2.0 * (torch.sqrt(dx * dx + dy * dy) - R) / cfg["W"])
        phi = torch.maximum(phi, p)
        u[0] += p * vx
        u[1] += p * vy
    return cfg, phi.float(), u.float(), torch.zeros_like(phi).float()


def _sim(cfg, fields, storage):
    sim = Sim(pfinputs.model_params(cfg), storage=storage)
    sim.init_fields(*fields)
    sim.release_work()
    return sim


def _ensemble(case, seed):
    return [_drops(case["n"], 1000 * seed + k) for k in range(case["domains"])]


def _net_inputs(case, seed):
    """Standardised fields, the density channel and the padding channels, BF16; the
    normalised residuals of a training target."""
    gen = torch.Generator().manual_seed(seed)
    B, H, W = case["batch"], case["H"], case["W"]
    dev = _device()
    x = torch.zeros((B, H, W, 8))
    x[..., :4] = torch.randn((B, H, W, 4), generator=gen)
    x[..., 4] = torch.rand((B, 1, 1), generator=gen) / 2.0 + 0.3
    y = torch.randn((B, H, W, 4), generator=gen) if case["what"] == "gradients" else None
    return x.to(dev, torch.bfloat16), None if y is None else y.to(dev)


def _layer_inputs(case, seed):
    gen = torch.Generator().manual_seed(seed)
    B, H, W, cin, cout = (case[k] for k in ("batch", "H", "W", "Cin", "Cout"))
    dev = _device()
    hin, win = {SAME: (H, W), UP: (H // 2, W // 2), POOL: (2 * H, 2 * W)}[case["mode"]]
    x = torch.nn.functional.silu(torch.randn((B, hin, win, cin), generator=gen))
    w = torch.randn((cout, 3, 3, cin), generator=gen) * math.sqrt(2.0 / (9 * cin))
    b = 0.01 * torch.randn((cout,), generator=gen)
    dy = torch.randn((B, H, W, cout), generator=gen)
    bf = torch.bfloat16
    return x.to(dev, bf), w.to(dev, bf), b.to(dev), dy.to(dev, bf)


def prepare(case, seed):
    what = case["what"]
    if what == "step":
        cfg = _config(case)
        return case, _sim(cfg, _fields(cfg, seed), case["storage"])
    if what == "ensemble":
        return case, [_sim(cfg, f, case["storage"]) for cfg, *f in _ensemble(case, seed)]
    if what == "layer":
        return case, _layer_inputs(case, seed)
    norm = dict(in_shift=[0.0] * 4, in_scale=[1.0] * 4, out_scale=[1.0] * 4, lrr_scale=1.0)
    sur = Surrogate(case["H"], case["W"], case["batch"], norm)
    sur.set_params(init_params(seed))
    return case, (sur,) + _net_inputs(case, seed)


def run(state):
    case, s = state
    what = case["what"]
    if what == "step":
        s.step(case["steps"])
        return s.read(("phi", "P", "J"))
    if what == "ensemble":
        Sim.step_many(s, case["steps"])
        out = [sim.read(("phi", "P", "J")) for sim in s]
        return {k: torch.stack([o[k] for o in out]) for k in ("phi", "P", "J")}
    if what == "forward":
        sur, x, _ = s
        return sur.forward(x)
    if what == "gradients":
        sur, x, y = s
        return sur.gradients(x, y)
    x, w, b, dy = s
    return conv_fwd(x, w, b, case["mode"]) + conv_wgrad(x, dy, case["mode"])


# ---------------------------------------------------------------------------
# the same results in float64
# ---------------------------------------------------------------------------
_C9 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (1, 1, 0), (-1, -1, 0),
       (1, -1, 0), (-1, 1, 0)]
_C19 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
        (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
        (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]


class _Lattice:
    """The method in float64 torch: fields (nz, ny, nx), populations as lists over the
    directions, T = 1/3."""

    def __init__(self, cfg):
        self.p = cfg
        self.c = _C9 if cfg["lattice"] == 9 else _C19
        self.D = 2 if cfg["lattice"] == 9 else 3
        rest, axis = (4 / 9, 1 / 9) if self.D == 2 else (1 / 3, 1 / 18)
        self.w = [(rest, axis, 1 / 36)[sum(abs(v) for v in c)] for c in self.c]
        self.wall = [b == pfinputs.WALL for b in cfg["bc"]]
        op = cfg.get("open_P")
        self.top = None if op is None else float(op[5])      # the open top's pressure

    def shift(self, f, c):
        """f(x + c), the adjacent site's value beyond a wall."""
        for a in range(3):
            if c[a] == 0:
                continue
            d = 2 - a
            g = torch.roll(f, -c[a], d)
            if self.wall[a]:
                at = f.shape[d] - 1 if c[a] > 0 else 0
                g.narrow(d, at, 1).copy_(f.narrow(d, at, 1))
            f = g
        return f

    def macros(self, phi, sg, jg, u=None, P=None):
        p = self.p
        grad = [torch.zeros_like(phi) for _ in range(3)]
        lap = torch.zeros_like(phi)
        for c, w in zip(self.c[1:], self.w[1:]):
            d = self.shift(phi, c)
            lap += 6.0 * w * (d - phi)
            for a in range(3):
                if c[a]:
                    grad[a] += 3.0 * w * c[a] * d
        m = dict(phi=phi, grad=grad, lap=lap)
        dr = p["rho_H"] - p["rho_L"]
        m["rho"] = p["rho_L"] + phi * dr
        it = [1.0 / (3.0 * p[k] + 0.5) for k in ("nu_L", "nu_H")]
        m["itau"] = it[0] + phi * (it[1] - it[0])
        m["mu"] = (48.0 * p["sigma"] / p["W"]) * phi * (phi - 1.0) * (phi - 0.5) \
            - 1.5 * p["sigma"] * p["W"] * lap
        gn = torch.sqrt(sum(g * g for g in grad))
        m["n"] = [g / (gn + p["eps"]) for g in grad]
        m["theta"] = 3.0 * p["M"] * (1.0 - 4.0 * (phi - 0.5) ** 2) / p["W"]
        m["F"] = [m["rho"] * g for g in p["g"]]
        if u is None:
            J = [j + 0.5 * (m["mu"] * g + F) for j, g, F in zip(jg, grad, m["F"])]
            rp = m["rho"] + (dr * lap / 4.0 if p["hoc"] else 0.0)
            u = [j / rp for j in J]
            P = sg / 3.0 + dr / 6.0 * sum(a * b for a, b in zip(u, grad))
            m["J"] = J
        m["u"], m["P"] = u, P
        return m

    def equilibrium(self, m, i):
        """h^eq, g^eq and K of direction i."""
        p, c, w = self.p, self.c[i], self.w[i]
        dr = p["rho_H"] - p["rho_L"]
        u, grad, F = m["u"], m["grad"], m["F"]

        def dot(v):
            return sum((c[a] * v[a] for a in range(3) if c[a]), torch.zeros_like(m["phi"]))

        cu = dot(u)
        gam = w * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * sum(v * v for v in u))
        heq = m["phi"] * gam + w * m["theta"] * dot(m["n"])
        K = ((gam - w) * dr + 3.0 * gam * m["mu"]) * (dot(grad) - sum(a * b for a, b in zip(u, grad))) \
            + 3.0 * gam * (dot(F) - sum(a * b for a, b in zip(u, F)))
        geq = m["rho"] * gam + w * (3.0 * m["P"] - m["rho"]) - 0.5 * K
        if p["hoc"]:
            geq = geq + 0.75 * w * cu * dr * m["lap"]
        return heq, geq, K

    def start(self, phi, u, P):
        m = self.macros(phi, None, None, u=list(u), P=P)
        eq = [self.equilibrium(m, i) for i in range(len(self.c))]
        return [e[0] for e in eq], [e[1] for e in eq]

    def look(self, h, g):
        jg = [sum((c[a] * v for c, v in zip(self.c, g) if c[a]), torch.zeros_like(h[0]))
              for a in range(3)]
        return self.macros(sum(h), sum(g), jg)

    def step(self, h, g):
        m = self.look(h, g)
        om = 1.0 / (3.0 * self.p["M"] + 0.5)
        eq = [self.equilibrium(m, i) for i in range(len(self.c))]
        Pi = {}
        for a in range(3):
            for b in range(a, 3):
                s = torch.zeros_like(h[0])
                for c, v, e in zip(self.c, g, eq):
                    if c[a] * c[b]:
                        s += c[a] * c[b] * (v - e[1])
                Pi[a, b] = s
        tr = (Pi[0, 0] + Pi[1, 1] + Pi[2, 2]) / 3.0
        hs, gs = [], []
        for i, (c, w) in enumerate(zip(self.c, self.w)):
            heq, geq, K = eq[i]
            cc = -tr
            for (a, b), v in Pi.items():
                if c[a] * c[b]:
                    cc = cc + (1.0 if a == b else 2.0) * c[a] * c[b] * v
            hs.append(h[i] + om * (heq - h[i]))
            gs.append(geq + K + (1.0 - m["itau"]) * 4.5 * w * cc)
        del eq
        return self.stream(hs, None), self.stream(gs, m["P"])

    def stream(self, f, P):
        out = []
        for i, c in enumerate(self.c):
            v = torch.roll(f[i], (c[2], c[1], c[0]), (0, 1, 2))
            back = f[i + 1 if i & 1 else i - 1] if i else f[0]
            if self.top is not None and c[2] < 0:
                # through the open top: the layer's own outgoing value at x - c_i put back
                # into the layer, and for g the pressure shift towards the top's
                enter = torch.roll(f[i][-1], (c[1], c[0]), (0, 1))
                if P is not None:
                    enter = enter + 6.0 * self.w[i] * (
                        self.top - torch.roll(P[-1], (c[1], c[0]), (0, 1)))
                v[-1] = enter
            for a in range(3):
                if c[a] and self.wall[a] and not (a == 2 and c[2] < 0 and self.top is not None):
                    at = 0 if c[a] > 0 else v.shape[2 - a] - 1
                    v.narrow(2 - a, at, 1).copy_(back.narrow(2 - a, at, 1))
            out.append(v)
        return out

    def run(self, fields, steps):
        phi, u, P = (t.double() for t in fields)
        h, g = self.start(phi, u, P)
        for _ in range(steps):
            h, g = self.step(h, g)
        m = self.look(h, g)
        return dict(phi=m["phi"], P=m["P"], J=torch.stack(m["J"][:self.D]))


def _conv(x, w, b=None):
    out = 0.0 if b is None else b
    for ky in range(3):
        for kx in range(3):
            out = out + torch.roll(x, (1 - ky, 1 - kx), (1, 2)) @ w[:, ky, kx, :].T
    return out


def _up(x):
    return x.repeat_interleave(2, 1).repeat_interleave(2, 2)


def _pool(x):
    return 0.25 * (x[:, ::2, ::2] + x[:, ::2, 1::2] + x[:, 1::2, ::2] + x[:, 1::2, 1::2])


def _network(flat, x):
    silu = torch.nn.functional.silu
    at, p = 0, {}
    for name, cin, cout in LAYERS:
        n = cout * 9 * cin
        p[name] = (flat[at:at + n].view(cout, 3, 3, cin), flat[at + n:at + n + cout])
        at += n + cout

    def layer(name, v):
        return silu(_conv(v, *p[name]))

    e0 = layer("e0b", layer("e0a", x))
    e1 = layer("e1b", layer("e1a", _pool(e0)))
    e2 = layer("e2b", layer("e2a", _pool(e1)))
    d = layer("u2", _up(layer("b3b", layer("b3a", _pool(e2)))))
    d = layer("d2b", layer("d2a", torch.cat([e2, d], 3)))
    d = layer("d1b", layer("d1a", torch.cat([e1, layer("u1", _up(d))], 3)))
    d = layer("d0b", layer("d0a", torch.cat([e0, layer("u0", _up(d))], 3)))
    n = HEAD[0] * HEAD[1]
    return d @ flat[at:at + n].view(HEAD[1], HEAD[0]).T + flat[at + n:]


def exact(case, seed):
    what = case["what"]
    if what == "step":
        cfg = _config(case)
        return _Lattice(cfg).run(_fields(cfg, seed), case["steps"])
    if what == "ensemble":
        # a flat lattice does not couple the layers of the third axis: one domain each
        every = _ensemble(case, seed)
        rho = torch.tensor([cfg["rho_H"] for cfg, *_ in every], dtype=torch.float64)
        cfg = dict(every[0][0], rho_H=rho.view(-1, 1, 1).to(_device()))
        out = _Lattice(cfg).run([torch.cat([e[k] for e in every], d)
                                 for k, d in ((1, 0), (2, 1), (3, 0))], case["steps"])
        return dict(phi=out["phi"].unsqueeze(1), P=out["P"].unsqueeze(1),
                    J=out["J"].transpose(0, 1).unsqueeze(2))
    if what == "layer":
        x, w, b, dy = (t.double() for t in _layer_inputs(case, seed))
        x = {SAME: lambda v: v, UP: _up, POOL: _pool}[case["mode"]](x)
        w.requires_grad_(True)
        pre = _conv(x, w, b)
        (dw,) = torch.autograd.grad(pre, w, dy)
        pre = pre.detach()
        return pre, torch.nn.functional.silu(pre), dw, dy.sum((0, 1, 2))
    x, y = _net_inputs(case, seed)
    flat = torch.from_numpy(np.asarray(init_params(seed))).to(x.device).double()
    if what == "forward":
        with torch.no_grad():
            return _network(flat, x.double())
    flat.requires_grad_(True)
    loss = ((_network(flat, x.double()) - y.double()) ** 2).mean()
    (grad,) = torch.autograd.grad(loss, flat)
    return grad, float(loss.detach())


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Stepping counts each step's state read once and written once (a step is the unit
    the method is made of) and the fields written by the read-out; the network's passes
    their inputs, parameters and outputs and the convolutions' products."""
    what = case["what"]
    if what in ("step", "ensemble"):
        flat = what == "ensemble" or case["nz"] == 1
        N = case["domains"] * case["n"] ** 2 if what == "ensemble" else \
            case["nx"] * case["ny"] * case["nz"]
        Q, D = (9, 2) if flat else (19, 3)
        site = 24 + 4 * (Q - 1) if case["storage"] == "fp16s" else 8 * Q
        return dict(bytes=N * (2 * site * case["steps"] + 4 * (2 + D)),
                    flops=N * case["steps"] * (400 if flat else 1000))
    P = case["batch"] * case["H"] * case["W"]
    if what == "layer":
        cin, cout = case["Cin"], case["Cout"]
        pin = {SAME: P, UP: P // 4, POOL: 4 * P}[case["mode"]]
        # x, dy, the pre-activation and the activation; forward and weight gradient
        return dict(bytes=2 * pin * cin + 2 * P * cout + 6 * P * cout + 4 * 9 * cin * cout,
                    flops=2 * 2 * P * 9 * cin * cout)
    level = {"0": 1, "1": 4, "2": 16, "3": 64}
    fwd = sum(2 * P * 9 * cin * cout / level[name[1]] for name, cin, cout in LAYERS) + \
        2 * P * HEAD[0] * HEAD[1]
    params = sum(9 * cin * cout + cout for _, cin, cout in LAYERS) + HEAD[1] * (HEAD[0] + 1)
    if what == "forward":
        return dict(bytes=P * 32 + 2 * params, flops=fwd)
    return dict(bytes=P * 32 + 6 * params, flops=3 * fwd)
