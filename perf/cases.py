"""Performance cases: the work that users of this solver have it do, through its
public entry points, from single steps of a small grid to the 4096^2 floodplain.

listed() names the cases, draw(rng) gives further ones of the same ranges,
prepare(case, seed) builds what a program holds before the call (the solver,
batch, nest or network with its inputs), run(state) makes one pass and returns
its outputs, exact(case, seed) computes the same outputs in plain 64-bit torch
where that is feasible, and work(case) states the bytes and operations one pass
cannot do without.

Kinds of case
  run       Solver.run(steps), then Solver.state(): a simulation advanced from
            one output frame to the next (it goes on from pass to pass)
  restart   Solver.set_state, set_time, run, state: a window re-run from a
            stored layer (checkpoints, data assimilation, the guarded run)
  noalloc   step_noalloc: one step of device tensors the caller owns
  batch     Batch.run, then the state of every scenario: the ensemble
  nest      Nest.run, then the coarse and patch states: zoomed-in areas
  learned   Solver.run of a coarse grid with the correction network attached
  fit       Net.fit: optimisation steps on the collected data set
  train     Net.train_step on host crops, then the gradient
"""
import math

import numpy as np
import torch

from paper_1705_00614_amd import learned as LC
from paper_1705_00614_amd import scenarios as S
from paper_1705_00614_amd import swe


def listed():
    return [
        # the smallest call: one step of a small grid and its frame, all latency
        dict(name="dam_128_one_step", kind="run", scene="dam", nx=128, ny=128, precision=32, limiter=0, steps=1),
        # the parity configuration (256^2 dam break, 200 FP64 steps), re-run
        # from its stored layer
        dict(name="dam_256_f64_restart", kind="restart", scene="dam", nx=256, ny=256, precision=64, limiter=0,
             steps=200),
        # the headline workload: a flood through the 4096^2 floodplain, few
        # tiles wet, between two output frames
        dict(name="flood_4096", kind="run", scene="flood", nx=4096, ny=4096, precision=32, limiter=0, steps=2000),
        # the same family in FP64 with the van Leer limiter, at the paper's 1024^2
        dict(name="flood_1024_f64_vanleer", kind="run", scene="flood", nx=1024, ny=1024, precision=64, limiter=1,
             steps=500),
        # fully wet control: most tiles listed, every stage at work
        dict(name="lake_2048", kind="run", scene="lake", nx=2048, ny=2048, precision=32, limiter=0, steps=200),
        # rain and losses on rough wet/dry ground, sides that are no multiple
        # of a tile, the monotonised central limiter
        dict(name="rain_1000x777", kind="run", scene="rain", nx=1000, ny=777, precision=32, limiter=2, steps=100),
        # one step of a caller's device layer, every tile, at the largest size
        dict(name="lake_4096_noalloc", kind="noalloc", scene="lake", nx=4096, ny=4096, precision=32, limiter=0),
        # an ensemble over hydrographs and gates, uneven sides
        dict(name="ensemble_20", kind="batch", n=20, side_min=256, side_max=1024, precision=32, steps=500),
        # two refined patches on the channel bends, with feedback
        dict(name="nest_512_r4", kind="nest", n=512, box=96, r=4, feedback=True, precision=32, steps=100),
        # a coarse grid corrected by the network before each step
        dict(name="learned_1024", kind="learned", n=1024, precision=32, steps=400),
        # training: optimisation steps on collected crops, and one on host crops
        dict(name="fit_b64", kind="fit", precision=32, batch=64, iters=16),
        dict(name="train_step_24", kind="train", tile=32, n=24),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "restart", "noalloc", "batch", "nest", "learned", "fit", "train"])
    lim = rng.choice([0, 0, 1, 2])
    if kind == "run":
        scene = rng.choice(["dam", "flood", "lake", "rain"])
        if scene == "flood":
            prec = rng.choice([32, 32, 64])
            n = _log(rng, 300, 3000 if prec == 32 else 1500)
            return dict(kind=kind, scene=scene, nx=n, ny=n, precision=prec, limiter=lim, steps=_log(rng, 100, 1500))
        prec = rng.choice([32, 32, 64])
        top = 2000 if prec == 32 and scene == "lake" else 900
        nx = _log(rng, 40, top)
        ny = nx if scene == "lake" else _log(rng, 40, top)
        return dict(kind=kind, scene=scene, nx=nx, ny=ny, precision=prec, limiter=lim, steps=_log(rng, 1, 200))
    if kind == "restart":
        return dict(kind=kind, scene=rng.choice(["dam", "rain"]), nx=_log(rng, 60, 600), ny=_log(rng, 60, 600),
                    precision=rng.choice([32, 64]), limiter=lim, steps=_log(rng, 20, 200))
    if kind == "noalloc":
        prec = rng.choice([32, 32, 64])
        n = _log(rng, 100, 4000 if prec == 32 else 2000)
        return dict(kind=kind, scene="lake", nx=n, ny=n, precision=prec, limiter=lim)
    if kind == "batch":
        lo = _log(rng, 100, 400)
        return dict(kind=kind, n=rng.randint(2, 20), side_min=lo, side_max=_log(rng, lo, 900),
                    precision=rng.choice([32, 32, 64]), steps=_log(rng, 50, 500))
    if kind == "nest":
        return dict(kind=kind, n=_log(rng, 256, 512), box=rng.randint(24, 64), r=rng.choice([2, 3, 4]),
                    feedback=rng.choice([True, True, False]), precision=rng.choice([32, 32, 64]),
                    steps=_log(rng, 10, 100))
    if kind == "learned":
        return dict(kind=kind, n=_log(rng, 200, 1000), precision=32, steps=_log(rng, 30, 400))
    if kind == "fit":
        return dict(kind=kind, precision=rng.choice([32, 64]), batch=rng.randint(5, 64), iters=rng.randint(4, 24))
    return dict(kind=kind, tile=rng.randint(4, 40), n=rng.randint(1, 24))


# ---------------------------------------------------------------- inputs

def _seed(seed):
    return int(seed) % (1 << 31)


def _scene(case, seed):
    """Scenario dict of a single-grid case."""
    rng = np.random.Generator(np.random.PCG64(_seed(seed)))
    nx, ny, prec, scene = case["nx"], case["ny"], case["precision"], case["scene"]
    if scene == "dam":
        sc = S.dam_break(nx, ny, x_dam=float(rng.uniform(0.3, 0.7)) * nx, h_left=float(rng.uniform(1.5, 3.0)),
                         h_right=float(rng.uniform(0.2, 0.8)), precision=prec)
    elif scene == "flood":
        sc = S.floodplain(n=nx, seed=_seed(seed), precision=prec, inlet_cells=min(40, nx // 8))
    elif scene == "lake":
        sc = S.floodplain_wet(n=nx, seed=_seed(seed), precision=prec)
        sc["params"].update(inlet=None, q_peak=0.0)
    else:   # rain over part of the area, losses over the rest
        sc = S.random_state(nx, ny, seed=_seed(seed), precision=prec)
        sc["sigma"] = np.where(S.fbm(ny, nx, 0.8, _seed(seed + 1), 1.0) > 0.5, 2e-5, -1e-5)
    sc["params"]["limiter"] = case["limiter"]
    return sc


def _ensemble(case, seed):
    """Scenarios of the ensemble family; the sides are the case's own, the rest is drawn."""
    rng = np.random.Generator(np.random.PCG64(case["n"] + 7919 * case["side_max"]))
    lo, hi = math.log(case["side_min"]), math.log(case["side_max"])
    sides = [int(round(math.exp(v))) for v in rng.uniform(lo, hi, size=case["n"])]
    return [S.ensemble(n=1, seed0=_seed(seed) + k, side_min=s, side_max=s, precision=case["precision"])[0]
            for k, s in enumerate(sides)]


def _crops(case, seed):
    """Host crops with labels and mask in the network's units, and weights."""
    rng = np.random.Generator(np.random.PCG64(_seed(seed)))
    n, so = case["n"], case["tile"] + 1
    x = rng.standard_normal((n, so + 8, so + 8, 6))
    x[..., 0] = np.maximum(x[..., 0], 0.0)
    x[..., 5] = x[..., 0] > 0.0
    x[..., 1:3] *= x[..., 5:]
    mask = (rng.uniform(size=(n, so, so, 6)) < 0.9).astype(np.float64)
    y = rng.standard_normal((n, so, so, 6)) * mask
    return x, y, mask, LC.initial_params(_seed(seed) + 1)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("run", "restart"):
        sc = _scene(case, seed)
        st = dict(case=case, g=swe.Solver(sc))
        if kind == "restart":
            st["layer"] = (sc["H0"], sc["Qx0"], sc["Qy0"])
        return st
    if kind == "noalloc":
        sc = _scene(case, seed)
        dt = torch.float32 if case["precision"] == 32 else torch.float64
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda").to(dt)
        b, H, Qx, Qy = (up(sc[k]) for k in ("b", "H0", "Qx0", "Qy0"))
        cf = up(sc["params"]["g"] * sc["n_manning"] ** 2)
        return dict(case=case, sc=sc, ins=(b, cf, H, Qx, Qy), outs=tuple(torch.empty_like(H) for _ in range(3)),
                    out=torch.empty(5, dtype=torch.float64, device="cuda"))
    if kind == "batch":
        return dict(case=case, b=swe.Batch(_ensemble(case, seed)))
    if kind == "nest":
        nd = S.nest_floodplain(n=case["n"], h=50.0, seed=_seed(seed), r=case["r"], box=case["box"],
                               precision=case["precision"])
        return dict(case=case, nest=swe.Nest(nd, feedback=case["feedback"]), patches=len(nd["patches"]))
    if kind == "learned":
        g = swe.Solver(S.floodplain(n=case["n"], h=100.0, seed=_seed(seed), t_peak=1800.0, sigma_t=600.0,
                                    inlet_cells=10, precision=case["precision"]))
        net = LC.make_net(g.work()["tile"][0], g.work()["ntiles"], out_scale=np.full(6, 0.02))
        net.set_params(LC.initial_params(_seed(seed)))
        net.attach(g)
        g.set_correction_depth(LC.CORR_DEPTH)
        return dict(case=case, g=g, net=net)
    if kind == "fit":
        fine = S.floodplain(n=768, h=25.0, seed=_seed(seed), t_peak=1800.0, sigma_t=600.0,
                            precision=case["precision"])
        net = LC.make_net(32 if case["precision"] == 32 else 16, 160)
        net.data(4096)
        LC.collect(net, fine, 4, 4, intervals=24, gap=8)
        net.set_out_scale(np.maximum(LC.label_scale(net), 1e-6))
        net.set_params(LC.initial_params(_seed(seed)))
        return dict(case=case, net=net, seed=_seed(seed))
    x, y, mask, p = _crops(case, seed)
    net = swe.Net(case["tile"], case["n"], np.ones(6), np.ones(6))
    net.set_params(p)
    return dict(case=case, net=net, data=(x, y, mask))


# ---------------------------------------------------------------- one pass

def _f32(a):
    """The network computes and stores FP32; its host copies widen it, and this
    is the same value in its own type."""
    return a.astype(np.float32)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "noalloc":
        swe.step_noalloc(state["sc"], *state["ins"], *state["outs"], 0.0, state["out"])
        return dict(zip(("H", "Qx", "Qy", "scalars"), (*state["outs"], state["out"])))
    if kind == "batch":
        b = state["b"]
        b.run(case["steps"])
        q = b.query()
        return dict(states=[b.state(k) for k in range(b.n)], time=q["time"], mass=q["mass"])
    if kind == "nest":
        n = state["nest"]
        n.run(case["steps"])
        return dict(coarse=n.coarse_state(), patches=[n.patch_state(k) for k in range(state["patches"])],
                    time=n.time())
    if kind == "fit":
        losses = state["net"].fit(case["iters"], case["batch"], 1e-3, seed=state["seed"])
        return dict(losses=_f32(losses), params=_f32(state["net"].params()), grads=_f32(state["net"].grads()))
    if kind == "train":
        loss = state["net"].train_step(*state["data"], 1e-3)
        return dict(loss=np.float32(loss), grads=_f32(state["net"].grads()))
    g = state["g"]
    if kind == "restart":
        g.set_state(*state["layer"])
        g.set_time(0.0)
    g.run(case["steps"])
    H, Qx, Qy = g.state()
    return dict(H=H, Qx=Qx, Qy=Qy, time=g.time())


# ---------------------------------------------------------------- floors

# channel cells across times the winding of the centre line, plus the flooded
# margin: wet cells of a floodplain of side n are about WET_PER_ROW * n
WET_PER_ROW = 14.0
CELL_FLOPS = 400.0   # of one cell and step, all four stages
NET_FLOPS = 2.0 * 9.0


def _net_flops(n, tile):
    """Multiply-adds of one forward of n crops, as operations."""
    so = tile + 1
    return n * sum(NET_FLOPS * ci * co * (so + 6 - 2 * l) ** 2 for l, (ci, co) in enumerate(swe.LC_LAYERS))


def work(case):
    kind = case["kind"]
    size = 8.0 if case.get("precision") == 64 else 4.0
    if kind in ("run", "restart", "noalloc"):
        cells = float(case["nx"]) * case["ny"]
        wet = {"dam": 1.0, "flood": min(1.0, WET_PER_ROW / case["nx"]), "lake": 0.6, "rain": 0.7}[case["scene"]]
        steps = case.get("steps", 1)
        step_bytes = steps * cells * wet * 8.0 * size
        host = 0.0 if kind == "noalloc" else cells * 3.0 * size * (2.0 if kind == "restart" else 1.0)
        return dict(bytes=max(step_bytes, 8.0 * size * cells if kind == "noalloc" else 0.0) + host,
                    flops=steps * cells * wet * CELL_FLOPS)
    if kind == "batch":
        mean = (case["side_max"] ** 2 - case["side_min"] ** 2) / (2.0 * math.log(case["side_max"] / case["side_min"])
                                                                  ) if case["side_max"] > case["side_min"] else \
            float(case["side_min"]) ** 2
        wet = case["n"] * WET_PER_ROW * math.sqrt(mean)
        return dict(bytes=case["steps"] * wet * 8.0 * size + case["n"] * mean * 3.0 * size,
                    flops=case["steps"] * wet * CELL_FLOPS)
    if kind == "nest":
        r, n, box = case["r"], case["n"], case["box"]
        wet = WET_PER_ROW / 2.0 * (n + 2.0 * r * r * r * box)
        return dict(bytes=case["steps"] * wet * 8.0 * size + (n * n + 2.0 * (r * box) ** 2) * 3.0 * size,
                    flops=case["steps"] * wet * CELL_FLOPS)
    if kind == "learned":
        n = float(case["n"])
        tiles = 3.0 * n / 32.0      # crops along the channel
        wet = 4.0 * n
        return dict(bytes=case["steps"] * wet * 8.0 * size + n * n * 3.0 * size,
                    flops=case["steps"] * (wet * CELL_FLOPS + _net_flops(tiles, 32)))
    tile = case["tile"] if kind == "train" else (32 if case["precision"] == 32 else 16)
    n = case["n"] if kind == "train" else case["batch"] * case["iters"]
    crop = 12.0 * (tile + 9) ** 2 + 2 * 24.0 * (tile + 1) ** 2
    return dict(bytes=n * crop + 12.0 * swe.load().swe_lc_nparams(), flops=3.0 * _net_flops(n, tile))


# ---------------------------------------------------------------- 64-bit values

def _pad(a, k, sx=1.0, sy=1.0):
    """k mirror images beyond each wall; the sign of a component normal to it flips."""
    a = torch.cat([sx * a[:, :k].flip(1), a, sx * a[:, -k:].flip(1)], 1)
    return torch.cat([sy * a[:k].flip(0), a, sy * a[-k:].flip(0)], 0)


def _at(p, k, dj, di):
    """The neighbour (dj, di) of every cell in an array padded by k."""
    return p[k + dj:p.shape[0] - k + dj, k + di:p.shape[1] - k + di]


def _minmod_like(lim, a, b):
    if lim == 1:
        m = 2.0 * a * b / torch.where(a * b > 0, a + b, torch.ones_like(a))
    elif lim == 2:
        m = torch.minimum(torch.minimum(2 * a.abs(), 2 * b.abs()), 0.5 * (a + b).abs()) * torch.sign(a)
    else:
        m = torch.where(a.abs() < b.abs(), a, b)
    return torch.where(a * b > 0, m, torch.zeros_like(a))


class _Exact:
    """The four-stage step of a walled grid in plain torch float64."""

    def __init__(self, sc):
        self.sc, self.p, self.h = sc, sc["params"], sc["h"]
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda")
        self.b, self.cf = up(sc["b"]), up(self.p["g"] * sc["n_manning"] ** 2)
        self.H = up(sc["H0"])
        wet = self.H > self.p["eps"]
        self.Qx, self.Qy = (torch.where(wet, up(sc[k]), torch.zeros_like(self.H)) for k in ("Qx0", "Qy0"))
        self.sigma = up(sc["sigma"]) if sc.get("sigma") is not None else None
        self.inlet = self.p.get("inlet")
        self.t = 0.0
        self.tau = self._cfl()

    def _vel(self, H, Qx, Qy):
        wet = H > self.p["eps"]
        Hs = torch.where(wet, H, torch.ones_like(H))
        z = torch.zeros_like(H)
        return wet, torch.where(wet, Qx / Hs, z), torch.where(wet, Qy / Hs, z)

    def _soft(self, H, wet, ux, uy):
        p = self.p
        wp = _pad(wet.double(), 1)
        xp, yp = _pad(ux, 1, -1.0, 1.0), _pad(uy, 1, 1.0, -1.0)
        vx, vy = torch.zeros_like(H), torch.zeros_like(H)
        for dj, di in ((0, -1), (0, 1), (-1, 0), (1, 0)):
            m = _at(wp, 1, dj, di)
            vx = vx + m * (_at(xp, 1, dj, di) - ux)
            vy = vy + m * (_at(yp, 1, dj, di) - uy)
        dx, dy = p["wind_x"] - ux, p["wind_y"] - uy
        k = p["wind_kappa"] * torch.sqrt(dx * dx + dy * dy) / H.clamp_min(p["h_wind"])
        nu = p["nu"] / self.h ** 2
        return nu * vx + p["f_cor"] * uy + k * dx, nu * vy - p["f_cor"] * ux + k * dy

    def _lam(self, H, wet):
        return self.cf / torch.where(wet, H, torch.ones_like(H)) ** (4.0 / 3.0)

    def _cfl(self):
        p = self.p
        wet, ux, uy = self._vel(self.H, self.Qx, self.Qy)
        fx, fy = self._soft(self.H, wet, ux, uy)
        fr = self._lam(self.H, wet) * torch.sqrt(ux * ux + uy * uy)
        fx, fy = fx - fr * ux, fy - fr * uy
        us = torch.maximum(ux.abs(), uy.abs()) + torch.sqrt(p["g"] * self.H)
        upx = (ux + torch.sign(fx) * torch.sqrt(self.h * fx.abs())).abs()
        upy = (uy + torch.sign(fy) * torch.sqrt(self.h * fy.abs())).abs()
        s = float(torch.where(wet, torch.maximum(us, torch.maximum(upx, upy)), torch.zeros_like(us)).max())
        tau = p["tau_max"] if p["tau_max"] > 0 else math.inf
        tau = min(tau, p["courant"] * self.h / s) if s > 0 else tau
        return min(tau, self.h ** 2 / (4 * p["nu"])) if p["nu"] > 0 else tau

    def _volume(self, tau):
        p = self.p
        v = p["q_base"] * tau
        if p["sigma_t"] > 0 and p["q_peak"] != p["q_base"]:
            k = 1.0 / (p["sigma_t"] * math.sqrt(2.0))
            v += (p["q_peak"] - p["q_base"]) * p["sigma_t"] * math.sqrt(math.pi / 2) * (
                math.erf((self.t + tau - p["t_peak"]) * k) - math.erf((self.t - p["t_peak"]) * k))
        return v

    def _faces(self, H, b, un, ut, axis):
        """Mass, normal and tangential flux through the faces across `axis`
        (H, b, un, ut padded by 2 along it): n + 1 faces."""
        g, eps, lim = self.p["g"], self.p["eps"], self.p["limiter"]
        n = H.shape[axis]
        lo = lambda a, k: a.narrow(axis, k, n - 2)
        wet = H > eps
        eta = H + b
        zero = torch.zeros_like(lo(H, 0))
        wm, wc, wq = (lo(wet, k) for k in range(3))
        sl = lambda a: _minmod_like(lim, lo(a, 1) - lo(a, 0), lo(a, 2) - lo(a, 1))
        slw = lambda a: _minmod_like(lim, torch.where(wm, lo(a, 1) - lo(a, 0), zero),
                                     torch.where(wq, lo(a, 2) - lo(a, 1), zero))
        side = {}
        for sgn in (1.0, -1.0):
            hf = 0.5 * sgn
            side[sgn] = (torch.where(wc, (lo(H, 1) + hf * sl(H)).clamp_min(0.0), zero),
                         torch.where(wc, lo(eta, 1) + hf * sl(eta), lo(b, 1)),
                         torch.where(wc, lo(un, 1) + hf * slw(un), zero),
                         torch.where(wc, lo(ut, 1) + hf * slw(ut), zero))
        L = [a.narrow(axis, 0, n - 3) for a in side[1.0]]
        R = [a.narrow(axis, 1, n - 3) for a in side[-1.0]]
        bs = torch.maximum(L[1] - L[0], R[1] - R[0])
        hL, hR = (L[1] - bs).clamp_min(0.0), (R[1] - bs).clamp_min(0.0)
        a = torch.maximum(L[2].abs() + torch.sqrt(g * hL), R[2].abs() + torch.sqrt(g * hR))
        qL, qR = hL * L[2], hR * R[2]
        return (0.5 * (qL + qR) - 0.5 * a * (hR - hL), 0.5 * (qL * L[2] + qR * R[2]) - 0.5 * a * (qR - qL),
                0.5 * (qL * L[3] + qR * R[3]) - 0.5 * a * (hR * R[3] - hL * L[3]))

    def step(self):
        p, tau, H, b = self.p, self.tau, self.H, self.b
        wet, ux, uy = self._vel(H, self.Qx, self.Qy)
        z = torch.zeros_like(H)
        dep = torch.where(wet, H, z)
        ec = b + dep
        dp, ep = _pad(dep, 1), _pad(ec, 1)
        e = {(j, i): torch.maximum(b, torch.minimum(_at(ep, 1, j, i), ec + _at(dp, 1, j, i)))
             for j in (-1, 0, 1) for i in (-1, 0, 1)}
        al = 1.0 / (12.0 * math.sqrt(2.0) - 14.0)
        be = (3.0 * math.sqrt(2.0) - 4.0) * al
        gx = (al * (e[0, 1] - e[0, -1]) + be * ((e[1, 1] - e[1, -1]) + (e[-1, 1] - e[-1, -1]))) / self.h
        gy = (al * (e[1, 0] - e[-1, 0]) + be * ((e[1, 1] - e[-1, 1]) + (e[1, -1] - e[-1, -1]))) / self.h
        lam = self._lam(H, wet)
        fx, fy = self._soft(H, wet, ux, uy)
        d = 1.0 + 0.5 * tau * lam * torch.sqrt(ux * ux + uy * uy)
        hx = torch.where(wet, (ux + 0.5 * tau * (fx - p["g"] * gx)) / d, z)
        hy = torch.where(wet, (uy + 0.5 * tau * (fy - p["g"] * gy)) / d, z)
        fx, fy = self._soft(H, wet, hx, hy)
        d = 1.0 + tau * lam * torch.sqrt(hx * hx + hy * hy)
        qx = torch.where(wet, H * (ux + tau * (fx - p["g"] * gx)) / d, z)
        qy = torch.where(wet, H * (uy + tau * (fy - p["g"] * gy)) / d, z)
        Ht = H.clone()
        vol = 0.0
        if self.inlet:
            i0, j0, ni, nj = self.inlet
            vol = self._volume(tau)
            Ht[j0:j0 + nj, i0:i0 + ni] += vol / (ni * nj * self.h ** 2)
        if self.sigma is not None:
            s = Ht + tau * self.sigma
            Ht = torch.where(self.sigma > 0, s, torch.where((self.sigma < 0) & wet, s.clamp_min(0.0), Ht))
        _, tx, ty = self._vel(Ht, qx, qy)
        px = lambda a, s: torch.cat([s * a[:, :2].flip(1), a, s * a[:, -2:].flip(1)], 1)
        py = lambda a, s: torch.cat([s * a[:2].flip(0), a, s * a[-2:].flip(0)], 0)
        xH, xN, xT = self._faces(px(Ht, 1), px(b, 1), px(tx, -1.0), px(ty, 1), 1)
        yH, yN, yT = self._faces(py(Ht, 1), py(b, 1), py(ty, -1.0), py(tx, 1), 0)
        r = tau / self.h
        Hn = Ht + r * (xH[:, :-1] - xH[:, 1:] + yH[:-1] - yH[1:])
        nx = qx + r * (xN[:, :-1] - xN[:, 1:] + yT[:-1] - yT[1:])
        ny = qy + r * (xT[:, :-1] - xT[:, 1:] + yN[:-1] - yN[1:])
        self.H = Hn.clamp_min(0.0)
        w = self.H > p["eps"]
        self.Qx, self.Qy = torch.where(w, nx, z), torch.where(w, ny, z)
        self.t += tau
        last = tau
        self.tau = self._cfl()
        return last, vol, float((self.H - Hn).sum()) * self.h ** 2


def _exact_net(case, seed):
    x, y, mask, p = _crops(case, seed)
    W, b = swe.lc_unpack(p)
    par = [torch.from_numpy(np.ascontiguousarray(a)).requires_grad_() for pair in zip(W, b) for a in pair]
    v = torch.from_numpy(x).permute(0, 3, 1, 2)
    for l in range(4):
        v = torch.nn.functional.conv2d(v, par[2 * l], par[2 * l + 1])
        v = torch.tanh(v) if l < 3 else v
    d = v.permute(0, 2, 3, 1) - torch.from_numpy(y)
    m = torch.from_numpy(mask)
    loss = 0.5 * (m * d * d).sum() / m.sum().clamp_min(1.0)
    loss.backward()
    return dict(loss=float(loss.detach()), grads=np.concatenate([a.grad.numpy().ravel() for a in par]))


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_net(case, seed)
    if kind not in ("run", "restart", "noalloc"):
        return None
    steps = case.get("steps", 1)
    if case["nx"] * case["ny"] * steps > 1.0e9 or steps > 600:   # over the time that a check can take
        return None
    g = _Exact(_scene(case, seed))
    for _ in range(steps):
        last, vol, clamped = g.step()
    if kind == "noalloc":
        return dict(H=g.H, Qx=g.Qx, Qy=g.Qy, scalars=None)
    out = [a.cpu().numpy() for a in (g.H, g.Qx, g.Qy)]
    return dict(H=out[0], Qx=out[1], Qy=out[2], time=g.t)
