"""Timed workloads of the library: what a user has it do, over the range of sizes it is used at.

Three kinds of pass, each through the package's Python binding:
  "step"   one capillary advanced by some steps, its fields read on the device
  "batch"  several capillaries advanced together, filled lengths sampled, fields read by the host
  "mlp"    the l(t) network: prediction (device or host arrays), loss gradient, training
Every case is a dict of plain values.  `exact` evaluates the same pass in FP64
with plain torch operations: the lattice Boltzmann step written literally
(populations, 9x9 change of basis, streaming by neighbour tables) and the
network with its gradients and Adam updates.
"""
import math

import numpy as np
import torch

from paper_0911_0459_amd import lbcap as L

# Model constants of the paper (Sec. 2 and Sec. 3.1) and, for the liquid-gas
# model, a mid level between the printed densities.
VDW = dict(kappa=0.02, a=9.0 / 49.0, b=2.0 / 21.0, T=0.56)
BIN = dict(kappa=0.04, A=0.04, B=0.04)
RHO_L, RHO_G = 4.54, 2.59
NU0 = 1.0 / 6.0


# ---- the cases ---------------------------------------------------------------------

def listed():
    return [
        # the smallest lattice the repository runs: the liquid-gas capillary of the
        # oracle gates, in the default launch configuration
        dict(name="vdw_256x64", kind="step", model="vdw", nx=256, ny=64, x_in=128, tube_len=128, tube_h=20, y0=22,
             steps=200, nu_l=0.1, nu_g=0.1, wall_grad=-0.144, Gamma=1.0, force=0.0, fp64=False, tuned=False),
        # channel flow driven by a body force (the Poiseuille check's setting), the
        # collision in FP64: walls along the whole lattice, odd sizes
        dict(name="bin_channel_force_fp64", kind="step", model="binary", nx=131, ny=41, x_in=0, tube_len=131,
             tube_h=39, y0=1, steps=200, nu_l=NU0, nu_g=NU0, wall_grad=0.0, Gamma=1.0, force=1e-5, fp64=True,
             tuned=False),
        # the liquid-gas capillary of the condensation study (700 x 40, L = 350): a
        # pitch that is no multiple of a wavefront
        dict(name="vdw_700x42", kind="step", model="vdw", nx=700, ny=42, x_in=175, tube_len=350, tube_h=40, y0=1,
             steps=200, nu_l=0.1, nu_g=0.1, wall_grad=-0.144, Gamma=1.0, force=0.0, fp64=False, tuned=False),
        # the binary capillary of the accuracy gates
        dict(name="bin_1024x128", kind="step", model="binary", nx=1024, ny=128, x_in=256, tube_len=768, tube_h=40,
             y0=44, steps=200, nu_l=NU0 * math.sqrt(10.0), nu_g=NU0 / math.sqrt(10.0), wall_grad=-0.2368,
             Gamma=1.0, force=0.0, fp64=False, tuned=False),
        # the binary throughput lattice
        dict(name="bin_4096x256", kind="step", model="binary", nx=4096, ny=256, x_in=1024, tube_len=3072, tube_h=100,
             y0=78, steps=100, nu_l=NU0 * math.sqrt(10.0), nu_g=NU0 / math.sqrt(10.0), wall_grad=-0.2368,
             Gamma=1.0, force=0.0, fp64=False, tuned=False),
        # a liquid-gas lattice far larger than the caches, launch shape tuned first
        dict(name="vdw_16384x1024", kind="step", model="vdw", nx=16384, ny=1024, x_in=4096, tube_len=12288,
             tube_h=400, y0=312, steps=32, nu_l=0.1, nu_g=0.1, wall_grad=-0.144, Gamma=1.0, force=0.0, fp64=False,
             tuned=True),
        # the mobility scan: one geometry, Gamma varied over a small batch, sampled
        dict(name="batch_mobility_5x512x64", kind="batch", model="binary", n=5, same=True, nx=512, ny=64,
             tube_len=384, tube_h=30, steps=200, every=100, ratio=1.0, theta=60.0, tuned=False),
        # the headline: a sweep of 256 uneven capillaries, tuned, sampled twice
        dict(name="batch_sweep_256", kind="batch", model="binary", n=256, same=False, nx=2506, ny=85, tube_len=2250,
             tube_h=45, steps=128, every=64, ratio=10.0, theta=60.0, tuned=True),
        # the network on one run (a gate decision), device arrays
        dict(name="mlp_predict_device_1", kind="mlp", do="predict_device", n=1),
        # the network on the held-out runs, host arrays
        dict(name="mlp_predict_507", kind="mlp", do="predict", n=507),
        # loss and gradient over the recorded training runs
        dict(name="mlp_loss_grad_3675", kind="mlp", do="loss_grad", n=3675),
        # one epoch of the ensemble's training
        dict(name="mlp_train_3675", kind="mlp", do="train", n=3675, batch=512, epochs=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.5:
        model = rng.choice(["vdw", "binary"])
        nodes = math.exp(rng.uniform(math.log(3e3), math.log(4e6)))
        ny = min(1024, max(16, int(math.sqrt(nodes / rng.uniform(2.0, 30.0)))))
        nx = min(16384, max(40, int(nodes / ny)))
        nu_l, nu_g = rng.uniform(0.08, 0.5), rng.uniform(0.08, 0.5)
        c = dict(kind="step", model=model, nx=nx, ny=ny, x_in=0, tube_len=0, tube_h=0, y0=0,
                 steps=int(min(250, max(16, 2e8 / nodes))), nu_l=nu_l, nu_g=nu_g if model == "binary" else nu_l,
                 wall_grad=-0.144 * rng.random() if model == "vdw" else rng.uniform(-0.35, 0.0),
                 Gamma=rng.uniform(0.25, 1.5), force=0.0, fp64=rng.random() < 0.15, tuned=rng.random() < 0.3)
        v = rng.random()
        if v < 0.1:      # no walls: a drop or a flat interface in a periodic box
            pass
        elif v < 0.2:    # a channel along the whole lattice, driven by a force
            c.update(tube_len=nx, tube_h=ny - 2, y0=1, force=1e-5 * rng.random())
        else:            # a capillary between reservoirs
            h = rng.randint(5, ny - 2)
            x_in = int(nx * rng.uniform(0.2, 0.5))
            c.update(x_in=x_in, tube_len=int((nx - x_in) * rng.uniform(0.5, 1.0)), tube_h=h,
                     y0=rng.randint(1, ny - 1 - h))
        return c
    if u < 0.65:
        n = _log_int(rng, 2, 24)
        ny = rng.randint(24, 160)
        nx = min(4000, max(200, int(4e6 / n / ny * rng.uniform(0.1, 1.0))))
        every = rng.randint(16, 50)
        return dict(kind="batch", model=rng.choice(["vdw", "binary", "binary"]), n=n, same=rng.random() < 0.5, nx=nx,
                    ny=ny, tube_len=int(nx * rng.uniform(0.4, 0.8)), tube_h=rng.randint(8, ny - 10), steps=2 * every,
                    every=every, ratio=math.exp(rng.uniform(0.0, math.log(30.0))), theta=rng.uniform(35.0, 85.0),
                    tuned=rng.random() < 0.3)
    do = rng.choice(["predict_device", "predict", "loss_grad", "train"])
    if do == "predict_device":
        return dict(kind="mlp", do=do, n=_log_int(rng, 1, 1024))
    if do == "train":
        return dict(kind="mlp", do=do, n=_log_int(rng, 100, 4000), batch=_log_int(rng, 48, 1024), epochs=1)
    return dict(kind="mlp", do=do, n=_log_int(rng, 1, 8192))


# ---- inputs ------------------------------------------------------------------------

def _wall_gradient(theta_deg):
    """Cahn's wall gradient of the binary model (A = B = kappa): cos(theta) =
    [(1 + w)^(3/2) - (1 - w)^(3/2)] / 2 with w = |G| sqrt(2)."""
    c = math.cos(math.radians(theta_deg))
    lo, hi = 0.0, 1.0
    for _ in range(80):
        w = 0.5 * (lo + hi)
        lo, hi = (w, hi) if 0.5 * ((1 + w) ** 1.5 - (1 - w) ** 1.5) < c else (lo, w)
    return -lo / math.sqrt(2.0)


def _capillaries(case, seed):
    """The pass's capillaries: (parameters, geometry, initial field) as plain values."""
    rng = np.random.default_rng(seed)
    vdw = case["model"] == "vdw"
    const = VDW if vdw else BIN
    liquid, gas, mid = (RHO_L, RHO_G, 0.5 * (RHO_L + RHO_G)) if vdw else (1.0, -1.0, 0.0)
    caps = []

    def add(g, p, l0):
        q = rng.random((g["ny"], g["nx"]))
        q *= 2e-3
        q += gas - 1e-3
        x = g["x_in"] if g["x_in"] > 0 else g["nx"] // 2
        q[:, x // 2: x] += liquid - gas
        if l0 and g["x_in"] > 0:   # the liquid column already in the tube
            q[g["y0"]: g["y0"] + g["tube_h"], x: x + l0] += liquid - gas
        caps.append((dict(const, model=case["model"], q_mid=mid, **p), g, q))

    if case["kind"] == "step":
        add({k: case[k] for k in ("nx", "ny", "x_in", "tube_len", "tube_h", "y0")},
            dict(nu_l=case["nu_l"], nu_g=case["nu_g"], wall_grad=case["wall_grad"], Gamma=case["Gamma"],
                 force_x=case["force"]), min(10, case["tube_len"]))
        return caps
    # batches: one geometry with the mobility varied, or sizes spread around the
    # given ones as the sweep of the repository spreads them; the sizes belong to
    # the case, only the fields come from the seed
    sizes = np.random.default_rng(4)
    for k in range(case["n"]):
        x_in = max(16, (case["nx"] - case["tube_len"]) * 3 // 4 if case["same"] else case["nx"] - case["tube_len"])
        if case["same"]:
            h, ln, ny, nx = case["tube_h"], case["tube_len"], case["ny"], case["nx"]
            ratio, theta, gamma = case["ratio"], case["theta"], 0.25 + 1.5 * k / max(1, case["n"] - 1)
        else:
            v = sizes.random(4)
            margin = case["ny"] - case["tube_h"]
            h = max(5, int(case["tube_h"] * (0.22 + 1.56 * v[0])))
            ln = max(32, int(case["tube_len"] * (0.22 + 1.56 * v[1])))
            ny, nx = h + margin, x_in + ln
            ratio, theta, gamma = case["ratio"] ** (2 * v[2]), case["theta"] + 40.0 * (v[3] - 0.5), 1.0
        g = dict(nx=nx, ny=ny, x_in=x_in, tube_len=ln, tube_h=h, y0=(ny - h) // 2)
        if vdw:
            p = dict(nu_l=0.1 + 0.02 * k / case["n"], nu_g=0.1, wall_grad=-0.144 * (1 + k) / case["n"])
            p["nu_g"] = p["nu_l"]
        else:
            p = dict(nu_l=NU0 * math.sqrt(ratio), nu_g=NU0 / math.sqrt(ratio), wall_grad=_wall_gradient(theta),
                     Gamma=gamma)
        add(g, p, 10)
    return caps


def _lb_params(p):
    return L.make_params(p["model"], **{k: v for k, v in p.items() if k != "model"})


DIMS = (19, 256, 256, 256, 64)


def _mlp_data(case, seed):
    """Parameters (trained-like scale: uniform within 1/sqrt(fan-in)), standardised
    features and targets, FP32."""
    rng = np.random.default_rng(seed)
    w = np.concatenate([rng.uniform(-1, 1, o * i + o) / math.sqrt(i) for i, o in zip(DIMS[:-1], DIMS[1:])])
    x = rng.standard_normal((case["n"], DIMS[0]))
    y = 0.5 * np.tanh(x @ rng.standard_normal((DIMS[0], DIMS[-1])) / 4.0) + 0.1 * rng.standard_normal((case["n"], DIMS[-1]))
    return w.astype(np.float32), x.astype(np.float32), y.astype(np.float32)


_compute = []


def _stream():
    """The program's one compute stream (a lattice steps from HIP graphs, which the
    default stream cannot capture)."""
    if not _compute:
        _compute.append(torch.cuda.Stream())
    return _compute[0].cuda_stream


def prepare(case, seed):
    if case["kind"] == "mlp":
        w, x, y = _mlp_data(case, seed)
        s = dict(case=case, net=L.MLP(seed=0), w=w, x=x, y=y)
        s["net"].set_params(w)
        if case["do"] == "predict_device":
            s["dx"] = torch.from_numpy(x).cuda()
            s["dy"] = torch.empty(case["n"], DIMS[-1], device="cuda")
        return s
    caps = _capillaries(case, seed)
    params = [_lb_params(p) for p, _, _ in caps]
    geoms = [L.make_geometry(**g) for _, g, _ in caps]
    fields = [q for _, _, q in caps]
    if case["kind"] == "step":
        lat = L.Lattice(params[0], geoms[0], fields[0], stream=_stream())
        if case["fp64"]:
            cfg = lat.launch_config()
            lat.set_launch_config(**dict(cfg.asdict(), fp64_arith=1))
    else:
        lat = L.Lattice(params, geoms, fields, stream=_stream())
    if case["tuned"]:
        lat.autotune(trial_steps=10)
    s = dict(case=case, lat=lat)
    # fields of capillary 0 on the device
    g = geoms[0]
    s["out"] = [torch.empty(g.ny, g.nx, device="cuda") for _ in range(4 if case["model"] == "binary" else 3)]
    torch.cuda.synchronize()
    return s


# ---- one pass ----------------------------------------------------------------------

def run(s):
    case = s["case"]
    if case["kind"] == "step":
        s["lat"].step(case["steps"])
        s["lat"].moments_device(*s["out"])
        return s["out"]
    if case["kind"] == "batch":
        lat = s["lat"]
        lat.step(case["steps"], sample_every=case["every"])
        lat.moments_device(*s["out"])
        health = lat.health()
        # l_eff(t) of every capillary, recorded in single precision as the
        # repository's recorder does; small batches read every capillary's fields
        res = dict(health=health, first=s["out"],
                   l_eff=np.stack([lat.l_history(k)[1] for k in range(case["n"])]).astype(np.float32))
        if case["n"] <= 8:
            res["fields"] = [np.stack(lat.moments(k)[: len(s["out"])]).astype(np.float32) for k in range(case["n"])]
        return res
    net = s["net"]
    if case["do"] == "predict_device":
        net.predict_device_noalloc(s["dx"], s["dy"])
        return s["dy"]
    if case["do"] == "predict":
        return net.predict(s["x"])
    if case["do"] == "loss_grad":
        loss, grad = net.loss_grad(s["x"], s["y"])
        return dict(loss=np.float32(loss), grad=grad)
    # a training from the given weights: upload, epochs, the trained weights back
    net.set_params(s["w"])
    loss = net.train(s["x"], s["y"], epochs=case["epochs"], batch=case["batch"], lr=1e-3, seed=5)
    return dict(loss=np.float32(loss), params=net.get_params())


def _nodes(case):
    """(fluid nodes, nodes) of all capillaries of a stepping case."""
    fluid = total = 0
    if case["kind"] == "step":
        total = case["nx"] * case["ny"]
        return total - case["tube_len"] * (case["ny"] - case["tube_h"]), total
    sizes = np.random.default_rng(4)
    for _ in range(case["n"]):
        if case["same"]:
            nx, ny, ln, h = case["nx"], case["ny"], case["tube_len"], case["tube_h"]
        else:
            v = sizes.random(4)
            h = max(5, int(case["tube_h"] * (0.22 + 1.56 * v[0])))
            ln = max(32, int(case["tube_len"] * (0.22 + 1.56 * v[1])))
            ny, nx = h + case["ny"] - case["tube_h"], max(16, case["nx"] - case["tube_len"]) + ln
        fluid += nx * ny - ln * (ny - h)
        total += nx * ny
    return fluid, total


def work(case):
    if case["kind"] != "mlp":
        # per step and fluid node: the nine populations (and phi) read and written
        # once, FP32; the fields of a capillary written once at the end
        fluid, _ = _nodes(case)
        per, flops = (72, 250) if case["model"] == "vdw" else (80, 420)
        return dict(bytes=float(fluid) * case["steps"] * per, flops=float(fluid) * case["steps"] * flops)
    w = sum(o * i + o for i, o in zip(DIMS[:-1], DIMS[1:]))
    macs = sum(o * i for i, o in zip(DIMS[:-1], DIMS[1:]))
    n, io = case["n"], DIMS[0] + DIMS[-1]
    if case["do"] in ("predict", "predict_device"):
        return dict(bytes=4.0 * (w + n * io), flops=2.0 * n * macs)
    grad_flops = 2.0 * n * (3 * macs - DIMS[0] * DIMS[1])
    if case["do"] == "loss_grad":
        return dict(bytes=4.0 * (2 * w + n * io), flops=grad_flops)
    steps = case["epochs"] * -(-n // case["batch"])
    return dict(bytes=4.0 * (6 * w * steps + case["epochs"] * n * io), flops=case["epochs"] * grad_flops)


# ---- the same passes in 64 bits ------------------------------------------------------

EX = (0, 1, -1, 0, 0, 1, -1, -1, 1)
EY = (0, 0, 0, 1, -1, 1, -1, 1, -1)
OPP = (0, 2, 1, 4, 3, 6, 5, 8, 7)
# rows of the change of basis of Appendix A: rho, e, eps, jx, qx, jy, qy, pxx, pxy
BASIS = ((1,) * 9, (-4, -1, -1, -1, -1, 2, 2, 2, 2), (4, -2, -2, -2, -2, 1, 1, 1, 1),
         (0, 1, -1, 0, 0, 1, -1, -1, 1), (0, -2, 2, 0, 0, 1, -1, -1, 1), (0, 0, 0, 1, -1, 1, -1, 1, -1),
         (0, 0, 0, -2, 2, 1, -1, 1, -1), (0, 1, 1, -1, -1, 0, 0, 0, 0), (0, 0, 0, 0, 0, 1, 1, -1, -1))
WEIGHT = (0.0,) + (1.0 / 3.0,) * 4 + (1.0 / 12.0,) * 4


def _tables(caps, dev):
    """Fluid nodes of all capillaries in one list: per direction the source of the
    streaming (an index into the 9 x N populations, bounce-back where the source
    is solid), and of the stencil value (an index into N, mirrored at walls)."""
    off, nodes, pulls, sten, wall = 0, [], [[] for _ in range(9)], [[] for _ in range(9)], [[] for _ in range(9)]
    per_node = [sum(g["nx"] * g["ny"] - g["tube_len"] * (g["ny"] - g["tube_h"]) for _, g, _ in caps)][0]
    for _, g, _ in caps:
        y, x = torch.meshgrid(torch.arange(g["ny"], device=dev), torch.arange(g["nx"], device=dev), indexing="ij")
        solid = (x >= g["x_in"]) & (x < g["x_in"] + g["tube_len"]) & ((y < g["y0"]) | (y >= g["y0"] + g["tube_h"]))
        fluid = ~solid.reshape(-1)
        ident = torch.cumsum(fluid, 0).reshape(g["ny"], g["nx"]) - 1 + off

        def at(t, dx, dy):   # t at r + (dx, dy)
            return torch.roll(t, (-dy, -dx), (0, 1)).reshape(-1)[fluid]

        own = ident.reshape(-1)[fluid]
        for i in range(9):
            ex, ey = EX[i], EY[i]
            src_solid = at(solid, -ex, -ey)
            pulls[i].append(torch.where(src_solid, OPP[i] * per_node + own, i * per_node + at(ident, -ex, -ey)))
            there = at(solid, ex, ey)
            if ex == 0 or ey == 0:
                ghost = at(ident, -ex, -ey)
            else:
                ghost = torch.where(at(solid, ex, 0), at(ident, -ex, ey),
                                    torch.where(at(solid, 0, ey), at(ident, ex, -ey), at(ident, -ex, -ey)))
            sten[i].append(torch.where(there, ghost, at(ident, ex, ey)))
            wall[i].append(there)
        nodes.append((off, fluid))
        off += int(own.numel())
    return nodes, [torch.cat(p) for p in pulls], [torch.cat(p) for p in sten], [torch.cat(p) for p in wall]


class _Exact:
    """Literal FP64 evaluation of the scheme on the fluid nodes of some capillaries."""

    def __init__(self, caps, dev):
        self.caps = caps
        self.vdw = caps[0][0]["model"] == "vdw"
        self.nodes, self.pull, self.sten, self.wall = _tables(caps, dev)
        count = [int(f.sum()) for _, f in self.nodes]
        rep = torch.tensor(count, device=dev)

        def per(key, default=0.0):
            v = [p.get(key, default) for p, _, _ in caps]
            if len(set(v)) == 1:
                return v[0]
            return torch.repeat_interleave(torch.tensor(v, dtype=torch.float64, device=dev), rep)

        self.G, self.nu_l, self.nu_g, self.Gamma = per("wall_grad"), per("nu_l"), per("nu_g"), per("Gamma", 1.0)
        self.force = per("force_x")
        self.p = caps[0][0]
        q = torch.cat([torch.from_numpy(f.reshape(-1)).to(dev)[m] for (_, _, f), (_, m) in zip(caps, self.nodes)])
        self.M = torch.tensor(BASIS, dtype=torch.float64, device=dev)
        self.Minv = torch.linalg.inv(self.M)
        self.bnd = self.wall[1].clone()
        for i in range(2, 9):
            self.bnd |= self.wall[i]
        self.free = (~self.bnd).double()
        zero = torch.zeros_like(q)
        self.rho = q if self.vdw else torch.ones_like(q)
        self.phi = zero if self.vdw else q
        self.ux = 0.5 * self.force * self.free / self.rho
        self.uy = zero
        # f = f^eq at rest, then the collision of time 0
        feq, _ = self.equilibrium(zero, zero)
        self.collide(feq)

    def stencil(self, q):
        v = [None] + [q[self.sten[i]] - 2.0 * self.G * self.wall[i] for i in range(1, 9)]
        dx = ((v[5] + v[8] - v[6] - v[7]) + 4.0 * (v[1] - v[2])) / 12.0
        dy = ((v[5] + v[7] - v[6] - v[8]) + 4.0 * (v[3] - v[4])) / 12.0
        lap = ((v[5] + v[6] + v[7] + v[8]) + 4.0 * (v[1] + v[2] + v[3] + v[4]) - 20.0 * q) / 6.0
        return dx, dy, lap

    def equilibrium(self, ux, uy):
        p, k = self.p, self.p["kappa"]
        q = self.rho if self.vdw else self.phi
        dx, dy, lap = self.stencil(q)
        if self.vdw:
            omega = 2.0 / (6.0 * self.nu_l + 1.0)
            r = self.rho
            p0 = r * p["T"] / (1.0 - p["b"] * r) - p["a"] * r * r
            base = 1.0 / 3.0 - (p["T"] / (1.0 - p["b"] * r) ** 2 - 2.0 * p["a"] * r)
            ls, lb = (1.0 / omega - 0.5) * base, 0.5 * base
            mu = None
        else:
            f = self.phi
            nu = self.nu_g + 0.5 * (f.clamp(-1.0, 1.0) + 1.0) * (self.nu_l - self.nu_g)
            omega = 2.0 / (6.0 * nu + 1.0)
            p0 = self.rho / 3.0 - 0.5 * p["A"] * f * f + 0.75 * p["B"] * f ** 4
            mu = -p["A"] * f + p["B"] * f ** 3 - k * lap
            ls = lb = 0.0
        X = p0 - k * q * lap
        udq = ux * dx + uy * dy
        qxx = self.rho * ux * ux + ls * (2.0 * ux * dx - udq) + 2.0 * lb * udq
        qyy = self.rho * uy * uy + ls * (2.0 * uy * dy - udq) + 2.0 * lb * udq
        qxy = self.rho * ux * uy + ls * (ux * dy + uy * dx)
        self.omega, self.mu = omega, mu
        feq = torch.empty(9, q.numel(), dtype=torch.float64, device=q.device)
        for i in range(1, 9):
            ex, ey, w = EX[i], EY[i], WEIGHT[i]
            quad = (ex * ex - 1.0 / 3.0) * qxx + (ey * ey - 1.0 / 3.0) * qyy + 2.0 * ex * ey * qxy
            if i <= 4:
                grad = (dx * dx / 3.0 - dy * dy / 6.0) if ex else (dy * dy / 3.0 - dx * dx / 6.0)
            else:
                grad = -(dx * dx + dy * dy) / 24.0 + 0.25 * ex * ey * dx * dy
            feq[i] = w * (X + self.rho * (ex * ux + ey * uy) + 1.5 * quad) + k * grad
        feq[0] = self.rho - feq[1:].sum(0)
        return feq, mu

    def collide(self, f):
        """Post-collision populations of the streamed f; self.ux, self.uy, rho, phi
        are those of f."""
        ux, uy = self.ux, self.uy
        feq, mu = self.equilibrium(ux, uy)
        m = self.M @ (f - feq)
        m[0] = 0.0
        m[3] = 0.0
        m[5] = 0.0
        # the force shifts u: j of f^eq is j + F/2; only the conserved rows see it
        # (zeroed above), and q_x, q_y relax fully
        m[7] = m[7] * self.omega
        m[8] = m[8] * self.omega
        post = f - self.Minv @ m
        if not (isinstance(self.force, float) and self.force == 0.0):
            F = self.force * self.free
            src = torch.zeros_like(f)
            for i in range(9):
                w = (4.0 / 9.0) if i == 0 else (1.0 / 9.0 if i <= 4 else 1.0 / 36.0)
                eu = EX[i] * ux + EY[i] * uy
                src[i] = w * (3.0 * (EX[i] - ux) + 9.0 * eu * EX[i]) * F
            s = self.M @ src
            s[1] *= 0.5
            s[2] *= 0.5
            s[4] *= 0.5
            s[6] *= 0.5
            s[7] = s[7] * (1.0 - 0.5 * self.omega)
            s[8] = s[8] * (1.0 - 0.5 * self.omega)
            post += self.Minv @ s
        self.f = post
        if not self.vdw:
            g = torch.empty_like(post)
            u2 = ux * ux + uy * uy
            for i in range(1, 9):
                eu = EX[i] * ux + EY[i] * uy
                g[i] = WEIGHT[i] * (self.Gamma * mu + self.phi * (eu + 1.5 * eu * eu - 0.5 * u2))
            g[0] = self.phi - g[1:].sum(0)
            self.g = g

    def step(self):
        flat = self.f.reshape(-1)
        f = torch.stack([flat[self.pull[i]] for i in range(9)])
        jx = sum(EX[i] * f[i] for i in range(1, 9))
        jy = sum(EY[i] * f[i] for i in range(1, 9))
        for i in range(1, 9):   # boundary nodes at rest
            f[i] -= WEIGHT[i] * (EX[i] * jx + EY[i] * jy) * self.bnd
        self.rho = f.sum(0)
        self.ux = (jx + 0.5 * self.force) * self.free / self.rho
        self.uy = jy * self.free / self.rho
        if not self.vdw:
            flat = self.g.reshape(-1)
            self.phi = sum(flat[self.pull[i]] for i in range(9))
        self.collide(f)

    def fields(self, k, count):
        off, fluid = self.nodes[k]
        n = int(fluid.sum())
        g = self.caps[k][1]
        res = []
        for q in (self.rho, self.ux, self.uy, self.phi)[:count]:
            t = torch.zeros(fluid.numel(), dtype=torch.float64, device=q.device)
            t[fluid] = q[off: off + n]
            res.append(t.reshape(g["ny"], g["nx"]))
        return res

    def l_eff(self):
        res = []
        for k, (p, g, _) in enumerate(self.caps):
            q = self.fields(k, 4)[0 if self.vdw else 3]
            h, y0, x0 = g["tube_h"], g["y0"], g["x_in"]
            rows = (y0 + h // 2 - 1, y0 + h // 2) if h % 2 == 0 else (y0 + h // 2, y0 + h // 2)
            line = (0.5 * (q[rows[0]] + q[rows[1]]))[x0: x0 + g["tube_len"]].cpu().numpy()
            below = np.nonzero(line < p["q_mid"])[0]
            if below.size == 0:
                l = float(g["tube_len"])
            elif below[0] == 0:
                l = 0.0
            else:
                j = int(below[0])
                l = j - 1 + (line[j - 1] - p["q_mid"]) / (line[j - 1] - line[j])
            res.append(l + 0.5 * h)
        return res


def _splitmix64(x):
    m = (1 << 64) - 1
    x = (x + 0x9E3779B97F4A7C15) & m
    x = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & m
    x = ((x ^ (x >> 27)) * 0x94D049BB133111EB) & m
    return x ^ (x >> 31)


def _net(w, x):
    h, o = x, 0
    for l, (i, j) in enumerate(zip(DIMS[:-1], DIMS[1:])):
        W, b = w[o: o + i * j].reshape(j, i), w[o + i * j: o + i * j + j]
        o += i * j + j
        h = h @ W.T + b
        if l < 3:
            h = 0.5 * h * (1.0 + torch.erf(h / math.sqrt(2.0)))
    return h


def _exact_mlp(case, seed, dev):
    w, x, y = (torch.from_numpy(a).to(dev).double() for a in _mlp_data(case, seed))
    if case["do"] in ("predict", "predict_device"):
        return _net(w, x)

    def grad(wv, xb, yb):
        wv = wv.detach().requires_grad_(True)
        loss = ((_net(wv, xb) - yb) ** 2).mean()
        return loss.detach(), torch.autograd.grad(loss, wv)[0]

    if case["do"] == "loss_grad":
        loss, g = grad(w, x, y)
        return dict(loss=loss, grad=g)
    # Adam over minibatches in the documented seeded order (Fisher-Yates on SplitMix64)
    n, batch = case["n"], case["batch"]
    m, v, t, last = torch.zeros_like(w), torch.zeros_like(w), 0, 0.0
    for e in range(case["epochs"]):
        perm = list(range(n))
        for i in range(n - 1, 0, -1):
            r = _splitmix64(((5 << 32) ^ ((e * 0x9E3779B97F4A7C15) & ((1 << 64) - 1)) ^ i) & ((1 << 64) - 1))
            j = r % (i + 1)
            perm[i], perm[j] = perm[j], perm[i]
        perm = torch.tensor(perm, device=dev)
        last = 0.0
        for b in range(0, n, batch):
            rows = perm[b: b + batch]
            loss, g = grad(w, x[rows], y[rows])
            last = last + loss * rows.numel()
            t += 1
            m = 0.9 * m + 0.1 * g
            v = 0.999 * v + 0.001 * g * g
            w = w - 1e-3 * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return dict(loss=last / n, params=w)


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if case["kind"] == "mlp":
        return _exact_mlp(case, seed, dev)
    caps = _capillaries(case, seed)
    e = _Exact(caps, dev)
    count = 3 if case["model"] == "vdw" else 4
    samples = []
    for t in range(1, case["steps"] + 1):
        e.step()
        if case["kind"] == "batch" and t % case["every"] == 0:
            samples.append(e.l_eff())
    if case["kind"] == "step":
        return e.fields(0, count)
    res = dict(health=None, first=e.fields(0, count), l_eff=np.array(samples).T.copy())
    if case["n"] <= 8:
        res["fields"] = [torch.stack(e.fields(k, count)) for k in range(case["n"])]
    return res
