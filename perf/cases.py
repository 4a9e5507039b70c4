"""The work that users of this library have it do, as timed cases.

Each case is one pass through the public entry points: a run of lattice steps
up to the next output (with the decoded fields), a network call, a training
step, a convolution layer both ways, the resistor network of a deposit, or the
analysis of a dried state.  ``listed`` names the cases, ``draw`` gives more of
the same ranges, ``exact`` the same outputs in 64 bits from plain torch.
"""
from __future__ import annotations

import ctypes as ct
import math

import numpy as np
import torch

from paper_2607_06794_amd import _lib, inputs
from paper_2607_06794_amd import surrogate as SU
from paper_2607_06794_amd.sim import Batch, Lattice, LatticeParams, kirchhoff

DEV = "cuda:0"
BYTES = {"f64": 8, "f32": 4, "f16dev": 2, "bf16dev": 2}
FIELD = {"f64": torch.float64, "f32": torch.float32, "f16dev": torch.float16, "bf16dev": torch.bfloat16}

# ghost pseudo-densities of the wall materials: the stripe and the rods wet A
PSI_SOLID = np.zeros((9, 2))
PSI_SOLID[inputs.STRIPE] = (0.60, 0.25)
PSI_SOLID[inputs.SURROUND] = (0.25, 0.60)
PSI_SOLID[inputs.ROD] = (0.60, 0.25)


def listed():
    return [
        # the static droplet of the parity runs: a small FP64 lattice, where
        # the launches and not the memory set the time
        {"name": "sphere_f64", "kind": "sphere", "prec": "f64", "n": 32, "steps": 50},
        # a small drying cap of odd extents, FP32, no rods
        {"name": "cap_ragged_f32", "kind": "cap", "prec": "f32", "nx": 117, "ny": 51, "nz": 37, "steps": 20},
        # the headline run: the full drying cap with 200 rods, FP32
        {"name": "cap_rods_f32", "kind": "rods", "prec": "f32", "nx": 256, "ny": 128, "nz": 64, "rods": 200,
         "steps": 20},
        # the full cap in half-precision storage with stochastic rounding
        {"name": "cap_f16", "kind": "cap", "prec": "f16dev", "nx": 256, "ny": 128, "nz": 64, "steps": 20},
        # the paper's colour-gradient fluid, full cap under a lid
        {"name": "cg_f32", "kind": "cg", "prec": "f32", "nx": 256, "ny": 128, "nz": 64, "steps": 10},
        # the paper's bead-spring filaments in the full cap
        {"name": "filaments_f32", "kind": "filaments", "prec": "f32", "nx": 256, "ny": 128, "nz": 64, "chains": 89,
         "steps": 10},
        # the parameter sweep: droplets of uneven size, stepped as one batch
        {"name": "sweep_batch", "kind": "batch", "prec": "f32", "first": 0, "count": 5, "steps": 10},
        # the surrogate's prediction on the full canvas
        {"name": "unet_predict", "kind": "predict", "D": 32, "H": 64, "W": 128},
        # one training step of the surrogate on one pair
        {"name": "unet_train", "kind": "train", "D": 32, "H": 64, "W": 128},
        # a decoder layer (upsampled input and skip) forward and backward
        {"name": "conv_layer", "kind": "conv", "D": 16, "H": 32, "W": 64, "c1": 128, "c2": 64, "cout": 64, "up": 1},
        # the resistor network of a dried deposit
        {"name": "network", "kind": "network", "rods": 300},
        # the analysis of a dried state at an output: masses, droplet shape,
        # deposit profiles, occupancy map, coarse canvas
        {"name": "analysis", "kind": "analysis", "prec": "f32", "nx": 256, "ny": 128, "nz": 64, "rods": 300},
    ]


def draw(rng):
    def span(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["sphere", "cap", "cap", "rods", "cg", "filaments", "batch", "predict", "train", "conv",
                       "network", "analysis"])
    if kind == "sphere":
        return {"kind": kind, "prec": rng.choice(["f64", "f32"]), "n": rng.randint(20, 32), "steps": rng.randint(5, 50)}
    if kind in ("predict", "train"):
        return {"kind": kind, "D": 8 * rng.randint(1, 4), "H": 8 * rng.randint(2, 8), "W": 8 * rng.randint(4, 16)}
    if kind == "conv":
        up = rng.randint(0, 1)
        return {"kind": kind, "D": 2 * rng.randint(2, 8), "H": 2 * rng.randint(3, 16), "W": 2 * rng.randint(4, 32),
                "c1": 8 * span(1, 16), "c2": 8 * span(1, 8) if up else 0, "cout": 8 * span(1, 8), "up": up}
    if kind == "network":
        return {"kind": kind, "rods": span(40, 300)}
    if kind == "batch":
        return {"kind": kind, "prec": "f32", "first": rng.randint(0, 40), "count": rng.randint(2, 4),
                "steps": rng.randint(2, 10)}
    nx, ny, nz = span(90, 256), span(50, 128), span(32, 64)
    c = {"kind": kind, "nx": nx, "ny": ny, "nz": nz}
    if kind == "cap":
        c.update(prec=rng.choice(["f32", "f16dev", "bf16dev"]), steps=rng.randint(4, 20))
    elif kind == "rods":
        c.update(prec="f32", rods=span(8, 200), steps=rng.randint(4, 20))
    elif kind == "cg":
        c.update(prec="f32", steps=rng.randint(3, 10))
    elif kind == "filaments":
        c.update(prec="f32", chains=span(4, 89), steps=rng.randint(3, 10))
    else:  # the coarse canvas takes even extents
        c.update(prec="f32", rods=span(20, 300), nx=nx & ~1, ny=ny & ~1, nz=nz & ~1)
    return c


# ---------------------------------------------------------------- inputs
def cap_spec(case, seed, reservoir=True):
    """The elongated cap of the benchmark at the case's extents."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    fx, fy = 0.586 * nx, 0.281 * ny
    return inputs.CapSpec(shape=(nz, ny, nx), footprint=(fx, fy), height=min(0.375 * nz, 0.67 * fy),
                          stripe=(min(round(fx + 10), nx), min(round(fy + 4), ny)), seed=seed, reservoir=reservoir)


def fluid_inputs(case, seed):
    """(rho0, material, LatticeParams) of a case's fluid."""
    kind, prec = case["kind"], case["prec"]
    if kind == "sphere":
        n = case["n"]
        rho, mat = inputs.sphere_droplet((n, n, n), n / 4, seed=seed)
        return rho, mat, LatticeParams(shape=(n, n, n), prec=prec, G=3.6, psi_solid=PSI_SOLID.copy())
    spec = cap_spec(case, seed, reservoir=kind != "cg")
    rho, mat = inputs.sessile_cap(spec)
    p = LatticeParams(shape=spec.shape, periodic=(True, True, False), prec=prec, G=3.6, psi_solid=PSI_SOLID.copy(),
                      evaporation=True)
    if prec in ("f16dev", "bf16dev"):
        p.rho_ref, p.rounding, p.sr_seed = (1.0, 1.0), "stochastic", 7
    if kind == "cg":
        mat[-1] = inputs.SURROUND
        rho[:, -1] = 0.0
        th = np.full(9, np.pi / 2)
        th[inputs.STRIPE], th[inputs.SURROUND] = np.deg2rad(60.0), np.deg2rad(120.0)
        p.evaporation, p.model, p.cg_sigma, p.cg_theta = False, "cg", 0.01, th
    return rho, mat, p


def with_rods(p, length=24.0, eps_att=1e-4):
    p.rod_length, p.rod_radius, p.rod_rho, p.eps_att, p.eps_rep = length, 2.0, 1.0, eps_att, 0.03
    p.rod_d0, p.rod_rcut, p.eps_wall, p.rod_d0_wall, p.n_sub, p.wall_z = 5.0, 7.5, 0.03, 3.0, 5, 0.5
    return p


def dried_rods(case, seed):
    """Rods lying crossed on the substrate over the benchmark deposit's region."""
    nx, ny = case["nx"], case["ny"]
    return inputs.deposit_rods(case["rods"], (0.156 * nx, 0.844 * nx), (4.0, ny - 4.0), 3.5, seed=seed)


def bead_positions(rods):
    """Beads every 2 nodes along each rod (L = 24, R = 2)."""
    q = rods[:, 3:7]
    axis = np.stack([2 * (q[:, 1] * q[:, 3] + q[:, 0] * q[:, 2]), 2 * (q[:, 2] * q[:, 3] - q[:, 0] * q[:, 1]),
                     1 - 2 * (q[:, 1] ** 2 + q[:, 2] ** 2)], axis=1)
    t = np.linspace(-10.0, 10.0, 11)
    return (rods[:, None, :3] + t[None, :, None] * axis[:, None, :]).reshape(-1, 3)


def circuit(case, seed):
    """(beads, x_src, x_snk) of a deposit of the benchmark's density: its
    region and electrode gap scale with the number of rods."""
    k = math.sqrt(case["rods"] / 300.0)
    rods = inputs.deposit_rods(case["rods"], (40.0 * k, 216.0 * k), (4.0 * k, 124.0 * k), 3.5, seed=seed)
    return bead_positions(rods), 68.0 * k, 188.0 * k


def chains(case, seed):
    """Straight chains of 12 beads at spacing 1.95 along x, on jittered places
    3 nodes apart inside the cap; at most case["chains"] of them."""
    rng = np.random.default_rng(seed)
    inside = inputs.cap_inside(cap_spec(case, seed))
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    half = 5.5 * 1.95
    places = [(x, y, z) for x in np.arange((nx - 1) / 2 % 26.0 - 26.0, nx, 26.0)
              for y in np.arange((ny - 1) / 2 % 3.0, ny, 3.0) for z in np.arange(2.6, nz, 3.0)
              if inside(x - half - 1, y, z + 1) and inside(x + half + 1, y, z + 1)]
    places = np.array(places)[rng.permutation(len(places))[:case["chains"]]]
    places = places + rng.uniform(-0.3, 0.3, places.shape)
    beads = places[:, None, :] + ((np.arange(12) - 5.5) * 1.95)[None, :, None] * np.array([1.0, 0.0, 0.0])
    return np.concatenate([beads.reshape(-1, 3), np.zeros((len(places) * 12, 3))], axis=1)


def canvases(case, seed):
    """A coarse canvas of a drying cap with rods, and one an interval later:
    smooth interface, velocities of 1e-3, rod fractions, mask."""
    D, H, W = case["D"], case["H"], case["W"]
    g = torch.Generator(device=DEV).manual_seed(seed)
    z, y, x = torch.meshgrid(*(torch.arange(n, device=DEV, dtype=torch.float32) for n in (D, H, W)), indexing="ij")
    out = []
    noise = torch.randn((5, D, H, W), generator=g, device=DEV)
    rod = (torch.rand((D, H, W), generator=g, device=DEV) < 0.03).float()
    drift = 0.97 + 0.02 * torch.rand((), generator=g, device=DEV)
    for k, s in enumerate((1.0, drift)):
        r = torch.sqrt(((x - W / 2 + 0.5) / (0.29 * W * s)) ** 2 + ((y - H / 2 + 0.5) / (0.2 * H)) ** 2
                       + (z / (0.4 * D * s)) ** 2)
        m = 0.5 - 0.5 * torch.tanh((r - 1) * 12)
        c = torch.zeros((D, H, W, 8), device=DEV)
        c[..., 0] = 0.03 + 0.97 * m + 1e-4 * noise[0]
        c[..., 1] = 1.0 - 0.97 * m + 1e-4 * noise[1]
        for a in range(3):
            c[..., 2 + a] = 2e-3 * noise[2 + a] * (1 - m) + 1e-3 * m * torch.sin(0.2 * (x + a * y + k))
        c[..., 5] = rod * m
        c[..., 6] = 1.0
        c[..., 7] = 1.0 - c[..., 5]
        c[:, :, W - W // 8:] = torch.tensor([0.03, 1, 0, 0, 0, 0, 0, 0], device=DEV)  # outside the lattice
        out.append(c.reshape(-1).contiguous())
    return out


def network_weights(net, seed):
    """Weights as a trained network has them: He-normal, small biases and output layer."""
    rng = np.random.default_rng(seed)
    host = np.zeros(net.nparam, np.float32)
    for name, c1, c2, co, _, _ in net.layers:
        o, nw, ob, nb = net.off[name]
        std = math.sqrt(2.0 / (27 * (c1 + c2))) * (0.3 if name == "out" else 1.0)
        host[o:o + nw] = rng.standard_normal(nw, dtype=np.float32) * std
        host[ob:ob + nb] = 0.02 * rng.standard_normal(nb, dtype=np.float32)
    return host


SCALE = np.array([0.05, 0.05, 1e-3, 1e-3, 1e-3, 0.02], np.float32)


def conv_inputs(case, seed):
    """BF16 operands of one layer: inputs, weights, and an upstream gradient."""
    D, H, W, c1, c2, co, up = (case[k] for k in ("D", "H", "W", "c1", "c2", "cout", "up"))
    g = torch.Generator(device=DEV).manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)
    x1 = torch.relu(rnd(D >> up, H >> up, W >> up, c1)).bfloat16()
    x2 = torch.relu(rnd(D, H, W, c2)).bfloat16() if c2 else None
    w = (rnd(27, c1 + c2, co) * math.sqrt(2.0 / (27 * (c1 + c2)))).bfloat16()
    b = 0.02 * rnd(co)
    dy = (1e-3 * rnd(D, H, W, co)).bfloat16().float()
    return x1, x2, w, b, dy


class State:
    """What a user's program holds between passes."""

    def __init__(self, case):
        self.case = case


def prepare(case, seed):
    s = State(case)
    kind = case["kind"]
    if kind in ("sphere", "cap", "cg"):
        rho, mat, p = fluid_inputs(case, seed)
        s.lat = Lattice(p, rho, mat)
        s.fields = field_buffers(s.lat)
    elif kind == "rods":
        rho, mat, p = fluid_inputs(case, seed)
        rods = inputs.place_rods(case["rods"], 24.0, 2.0, (case["nx"], case["ny"], case["nz"]), seed=seed,
                                 max_trials=4 * case["rods"])
        s.lat = Lattice(with_rods(p), rho, mat, rods=rods)
        s.fields = field_buffers(s.lat)
        s.snap = s.lat.snapshot()
    elif kind == "filaments":
        rho, mat, p = fluid_inputs(case, seed)
        beads = chains(case, seed)
        p.n_fil, p.fil_beads, p.wall_z, p.fil_eps_coh = len(beads) // 12, 12, 0.5, 4e-3
        s.lat = Lattice(p, rho, mat, beads=beads)
        s.fields = field_buffers(s.lat)
        s.snap = s.lat.snapshot()
    elif kind == "batch":
        s.lats, s.fields, s.snaps = [], [], []
        for d in inputs.sweep_droplets(case["first"] + case["count"], first=case["first"], run=seed + 1):
            p = LatticeParams(shape=d["shape"], periodic=(True, True, False), prec=case["prec"], G=3.6,
                              psi_solid=PSI_SOLID.copy(), evaporation=True)
            s.lats.append(Lattice(with_rods(p, d["rod_length"], d["eps_att"]), d["rho"], d["mat"], rods=d["rods"]))
            s.fields.append(field_buffers(s.lats[-1]))
        s.batch = Batch(s.lats)
        s.snaps = [lat.snapshot() for lat in s.lats]
    elif kind in ("predict", "train"):
        s.net = SU.UNet(case["D"], case["H"], case["W"])
        s.net.set_flat(network_weights(s.net, seed))
        s.net.set_scale(SCALE)
        s.x, s.tgt = canvases(case, seed)
        s.pred = torch.empty_like(s.x)
    elif kind == "conv":
        s.x1, s.x2, s.w, s.b, s.dy = conv_inputs(case, seed)
        D, H, W, cin, co = case["D"], case["H"], case["W"], case["c1"] + case["c2"], case["cout"]
        s.wt = torch.empty(co * 27 * cin, dtype=torch.bfloat16, device=DEV)
        s.y = torch.empty((D, H, W, co), dtype=torch.bfloat16, device=DEV)
        s.g = torch.empty_like(s.y)
        s.acc = torch.empty((D, H, W, co), dtype=torch.float32, device=DEV)
        s.dx = torch.empty((D, H, W, cin), dtype=torch.float32, device=DEV)
        s.dw = torch.empty((27, cin, co), dtype=torch.float32, device=DEV)
        s.db = torch.empty(co, dtype=torch.float32, device=DEV)
        s.lib, s.stream = _lib.load(), ct.c_void_p(torch.cuda.current_stream().cuda_stream)
        _lib.check(s.lib.lb_conv_pack_weights(ptr(s.w), cin, co, ptr(s.wt), s.stream))
        cv = s.conv = _lib.LbConv()
        cv.x1, cv.c1, cv.up1, cv.c2 = s.x1.data_ptr(), case["c1"], case["up"], case["c2"]
        cv.x2 = s.x2.data_ptr() if s.x2 is not None else None
        cv.w, cv.wt, cv.b, cv.y, cv.yf, cv.acc = (s.w.data_ptr(), s.wt.data_ptr(), s.b.data_ptr(), s.y.data_ptr(), None,
                                                  s.acc.data_ptr())
        cv.D, cv.H, cv.W, cv.cout, cv.relu = D, H, W, co, 1
    elif kind == "network":
        pos, s.src, s.snk = circuit(case, seed)
        s.pos = torch.from_numpy(pos).to(DEV)
    elif kind == "analysis":
        rho, mat, p = fluid_inputs(case, seed)
        s.lat = Lattice(with_rods(p), rho, mat, rods=dried_rods(case, seed))
        s.cells = tuple(-(-n // 16) * 8 for n in (case["nz"], case["ny"], case["nx"]))
    return s


def ptr(t):
    return ct.c_void_p(t.data_ptr())


def field_buffers(lat):
    """Device arrays for the decoded densities and populations of a lattice."""
    nz, ny, nx = lat.params.shape
    return (torch.empty((2, nz, ny, nx), dtype=torch.float64, device=DEV),
            torch.empty((2, 19, nz, ny, nx), dtype=torch.float64, device=DEV))


def fields(lat, bufs):
    """The lattice's decoded state on the device, in its storage type."""
    rho, f = bufs
    _lib.check(lat.lib.lb_export(lat._ctx, ptr(rho), ptr(f), ct.c_void_p(torch.cuda.current_stream().cuda_stream)))
    t = FIELD[lat.params.prec]
    return {"rho": rho.to(t), "f": f.to(t)}


def rod_table(lat):
    """The rods of one lattice of a sweep, in a table of the largest count."""
    out = np.zeros((400, 13), np.float32)
    out[:lat.n_rods] = lat.rods()
    return out


# ---------------------------------------------------------------- one pass
def run(s):
    case, kind = s.case, s.case["kind"]
    if kind in ("sphere", "cap", "cg"):
        s.lat.step(case["steps"])
        return fields(s.lat, s.fields)
    if kind == "rods":  # a branch from a saved state, up to its next output
        s.lat.restore(s.snap)
        s.lat.coupled_step(case["steps"])
        return {**fields(s.lat, s.fields), "rods": s.lat.rods().astype(np.float32)}
    if kind == "filaments":
        s.lat.restore(s.snap)
        s.lat.coupled_step(case["steps"])
        return {**fields(s.lat, s.fields), "beads": s.lat.beads().astype(np.float32)}
    if kind == "batch":
        for lat, snap in zip(s.lats, s.snaps):
            lat.restore(snap)
        s.batch.step(case["steps"], rods=True, graph=True)
        return [{**fields(lat, b), "rods": rod_table(lat)} for lat, b in zip(s.lats, s.fields)]
    if kind == "predict":
        SU.predict(s.net, s.x, pred_f32=s.pred)
        return {"pred": s.pred, "out": s.net.out}
    if kind == "train":  # an update of the rate's warm-up
        loss = s.net.train_step(None, s.x, s.tgt, lam=100.0, lr=3e-6)
        return {"loss": np.array(loss, np.float32), "g": s.net.g, "p": s.net.p, "out": s.net.out}
    if kind == "conv":
        n = s.y.numel()
        _lib.check(s.lib.lb_conv3d_forward(ct.byref(s.conv), s.stream))
        _lib.check(s.lib.lb_relu_grad(ptr(s.dy), ptr(s.y), n, 1, ptr(s.g), s.stream))
        _lib.check(s.lib.lb_conv3d_backward_data(ct.byref(s.conv), ptr(s.g), ptr(s.dx), s.stream))
        _lib.check(s.lib.lb_fill_f32(ptr(s.dw), s.dw.numel(), 0.0, s.stream))
        _lib.check(s.lib.lb_fill_f32(ptr(s.db), s.db.numel(), 0.0, s.stream))
        _lib.check(s.lib.lb_conv3d_backward_weights(ct.byref(s.conv), ptr(s.g), ptr(s.dw), ptr(s.db), s.stream))
        return {"y": s.y, "dx": s.dx, "dw": s.dw, "db": s.db}
    if kind == "network":
        r = kirchhoff(s.pos, 5.25, s.src, s.snk)
        return {k: r[k] for k in ("V", "I", "I_tot", "I_ref", "kappa", "edges", "n_source", "n_sink", "max_degree")}
    nx, ny = case["nx"], case["ny"]
    xc, yc = (nx - 1) / 2, (ny - 1) / 2
    o = s.lat.observables()
    d = s.lat.deposit(16, 8, xc, yc, float(nx), ny / 2.0, x_src=0.27 * nx, x_snk=0.73 * nx)
    canvas, _ = SU.restrict(s.lat, *s.cells)
    return {"mass": o["mass"], "kinetic": o["kinetic"], "fluid_nodes": o["fluid_nodes"], "status": o["status"],
            "shape": s.lat.droplet_shape(xc, yc), "deposit": d, "map": s.lat.rod_map(), "canvas": canvas}


# ---------------------------------------------------------------- the work
def layer_flops(case):
    n0 = case["D"] * case["H"] * case["W"]
    return sum(2.0 * 27 * (c1 + c2) * co * (n0 >> (3 * lvl)) for _, c1, c2, co, _, lvl in SU.layer_shapes())


def layer_bytes(case):
    """Inputs, weights and outputs of every layer once, BF16."""
    n0 = case["D"] * case["H"] * case["W"]
    return sum(2.0 * ((n0 >> (3 * lvl)) * ((c1 >> (3 * up)) + c2 + co) + 27 * (c1 + c2) * co)
               for _, c1, c2, co, up, lvl in SU.layer_shapes())


def work(case):
    kind = case["kind"]
    if kind == "predict":
        return {"bytes": layer_bytes(case), "flops": layer_flops(case)}
    if kind == "train":
        params = sum(27 * (c1 + c2) * co + co for _, c1, c2, co, _, _ in SU.layer_shapes())
        return {"bytes": 3 * layer_bytes(case) + 30 * params, "flops": 3 * layer_flops(case)}
    if kind == "conv":
        n, cin, co = case["D"] * case["H"] * case["W"], case["c1"] + case["c2"], case["cout"]
        x = (n >> (3 * case["up"])) * case["c1"] + n * case["c2"]
        return {"bytes": 2.0 * (2 * x + 2 * n * co + 2 * 27 * cin * co) + 4.0 * (n * co + n * cin + 27 * cin * co),
                "flops": 3 * 2.0 * 27 * cin * co * n}
    if kind == "network":
        n = 11 * case["rods"]
        # one sparse product of about 16 neighbours a bead per iteration
        return {"bytes": 24.0 * n + 16.0 * n, "flops": 250 * n * (2.0 * 16 + 12)}
    if kind == "batch":
        nodes = 0
        for i in range(case["first"], case["first"] + case["count"]):
            nx = (128, 160, 192, 224, 256)[i % 5]
            nodes += nx * (nx // 2) * (48 + 16 * (nx - 128) // 128)
    elif kind == "sphere":
        nodes = case["n"] ** 3
    else:
        nodes = case["nx"] * case["ny"] * case["nz"]
    state = 38.0 * nodes * BYTES[case["prec"]]
    if kind == "analysis":
        return {"bytes": 3 * state, "flops": 300.0 * nodes}
    steps = case["steps"]
    out = state + 40.0 * nodes * 8  # the decoded fields
    back = 0.0 if kind in ("sphere", "cap", "cg") else 2 * state  # the saved state
    return {"bytes": 2 * state * steps + out + back, "flops": 1100.0 * nodes * steps}


# ---------------------------------------------------------------- in 64 bits
C = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0), (1, -1, 0),
     (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]
Wt = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
OPP = [C.index((-c[0], -c[1], -c[2])) for c in C]


def at(a, c, sign=1):
    """a(x + sign c) on the periodic lattice (last three axes z, y, x)."""
    return torch.roll(a, shifts=(-sign * c[2], -sign * c[1], -sign * c[0]), dims=(-3, -2, -1))


def stencil(a):
    """sum_i w_i a(x + c_i) c_i per axis."""
    g = [0.0, 0.0, 0.0]
    for w, c in zip(Wt[1:], C[1:]):
        v = w * at(a, c)
        for d in range(3):
            if c[d]:
                g[d] = g[d] + v * c[d]
    return torch.stack(g)


def pull(f, mat, top):
    """The populations streamed into every node; walls return them halfway."""
    out = torch.empty_like(f)
    for i, c in enumerate(C):
        m = at(mat, c, -1)
        for k in range(2):
            v = torch.where(m >= 2, f[k, OPP[i]], at(f[k, i], c, -1))
            out[k, i] = torch.where(m == 1, torch.full_like(v, Wt[i] * top[k]), v)
    return out


def momentum(f):
    return torch.stack([sum(f[i] * c[d] for i, c in enumerate(C) if c[d]) for d in range(3)])


def equilibrium(rho, u, i):
    cu = C[i][0] * u[0] + C[i][1] * u[1] + C[i][2] * u[2]
    return Wt[i] * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * (u * u).sum(0))


def shan_chen(f, mat, fluid, G, top):
    """One step of the two-component pseudopotential fluid, tau = 1."""
    f = pull(f, mat, top)
    rho = f.sum(1)
    j = momentum(f[0]) + momentum(f[1])
    wall = torch.as_tensor(PSI_SOLID, device=f.device)[mat.long()]
    psi = [torch.where(fluid, rho[k], torch.where(mat == 1, torch.full_like(rho[k], top[k]), wall[..., k]))
           for k in range(2)]
    u = j / torch.where(fluid, rho[0] + rho[1], torch.ones_like(rho[0]))
    for k in range(2):
        F = -G * psi[k] * stencil(psi[1 - k])
        ok = fluid & (rho[k] >= 1e-12)
        ueq = u + torch.where(ok, F / torch.where(ok, rho[k], torch.ones_like(u[0])), torch.zeros_like(F))
        for i in range(19):
            f[k, i] = torch.where(fluid, equilibrium(rho[k], ueq, i), torch.zeros_like(u[0]))
    return f


def colour_gradient(f, mat, fluid, sigma, beta, theta):
    """One step of the colour-gradient fluid between static walls, tau = 1."""
    zero, one = torch.zeros_like(f[0, 0]), torch.ones_like(f[0, 0])
    f = pull(f, mat, (0.0, 0.0))
    rho = torch.where(fluid, f.sum(1), zero)
    r = torch.where(fluid, rho[0] + rho[1], one)
    col = (rho[0] - rho[1]) / r
    solid = mat >= 2
    num, den, cts = zero.clone(), zero.clone(), zero.clone()
    ct = torch.cos(torch.as_tensor(theta, device=f.device))[mat.long()] * solid
    for w, c in zip(Wt[1:], C[1:]):
        num, den, cts = num + w * at(col * fluid, c), den + w * at(fluid.double(), c), cts + w * at(ct, c)
    grad = 3 * stencil(torch.where(fluid, col, num / torch.where(den > 0, den, one))) * fluid
    mag = (grad * grad).sum(0).sqrt()
    has = fluid & (mag > 1e-2)
    n = torch.where(has, grad / torch.where(has, mag, one), zero)
    s = stencil(solid.double())
    ws = 1 - 1 / 3 - den
    near = fluid & (ws > 1e-9)
    nw = -s / torch.where(near & ((s * s).sum(0) > 0), (s * s).sum(0).sqrt(), one)
    cosw = cts / torch.where(near, ws, one)
    t = n - (n * nw).sum(0) * nw
    tm = (t * t).sum(0).sqrt()
    use = near & has & (tm > 1e-12)
    turned = -cosw * nw + (1 - cosw * cosw).clamp(min=0).sqrt() * t / torch.where(use, tm, one)
    n = torch.where(use, turned, n)
    div = zero.clone()
    for w, c in zip(Wt[1:], C[1:]):
        v = torch.where(at(has, c), at(n, c), n)
        div = div + w * (v[0] * c[0] + v[1] * c[1] + v[2] * c[2])
    F = 0.5 * sigma * (-3 * div) * mag * n * fluid
    u = (momentum(f[0]) + momentum(f[1]) + 0.5 * F) / r
    uF = (u * F).sum(0)
    out = torch.empty_like(f)
    seg = beta * rho[0] * rho[1] / r
    for i, c in enumerate(C):
        cu, cF = (sum(c[d] * v[d] for d in range(3)) + zero for v in (u, F))
        total = equilibrium(rho[0] + rho[1], u, i) + 0.5 * Wt[i] * (3 * (cF - uF) + 9 * cu * cF)
        cn = sum(c[d] * n[d] for d in range(3)) / max(1.0, math.sqrt(sum(v * v for v in c))) + zero
        for k in range(2):
            out[k, i] = torch.where(fluid, rho[k] / r * total + (1 - 2 * k) * seg * Wt[i] * cn, zero)
    return out


def conv64(x, w, b):
    """3 x 3 x 3 convolution, zero padding, channels last: tap by tap."""
    D, H, W, _ = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    y = b.expand(D * H * W, -1)
    for t in range(27):
        z, r, q = t // 9, t // 3 % 3, t % 3
        y = y + xp[z:z + D, r:r + H, q:q + W].reshape(D * H * W, -1) @ w[t]
    return y.reshape(D, H, W, -1)


def up64(x):
    for d in range(3):
        x = x.repeat_interleave(2, dim=d)
    return x


def unet64(x, weights):
    """The encoder-decoder on [D][H][W][8]; weights: name -> (w, b)."""
    skips, ch = [], SU.CH
    for lvl in range(len(ch)):
        for part in "ab":
            x = torch.relu(conv64(x, *weights["enc%d%s" % (lvl, part)]))
        if lvl < len(ch) - 1:
            skips.append(x)
            D, H, W, c = x.shape
            x = x.reshape(D // 2, 2, H // 2, 2, W // 2, 2, c).mean(dim=(1, 3, 5))
    for lvl in range(len(ch) - 2, -1, -1):
        x = torch.cat([up64(x), skips[lvl]], dim=-1)
        for part in "ab":
            x = torch.relu(conv64(x, *weights["dec%d%s" % (lvl, part)]))
    return conv64(x, *weights["out"])


def exact_network(case, seed, training):
    """The same network, weights and normalised input as held in BF16, all else in 64 bits."""
    net = SU.UNet(case["D"], case["H"], case["W"])  # its layout of the parameters alone
    host = torch.from_numpy(network_weights(net, seed)).to(DEV)
    weights, parts = {}, {}
    for name, c1, c2, co, _, _ in net.layers:
        o, nw, ob, nb = net.off[name]
        w = host[o:o + nw].bfloat16().double().reshape(27, c1 + c2, co).requires_grad_(training)
        b = host[ob:ob + nb].double().requires_grad_(training)
        weights[name], parts[name] = (w, b), (o, nw, ob, nb)
    x, tgt = (c.double().reshape(case["D"], case["H"], case["W"], 8) for c in canvases(case, seed))
    gain = torch.tensor([1, 1, 100, 100, 100, 1, 1, 1], dtype=torch.float64, device=DEV)
    out = unet64((x * gain).bfloat16().double(), weights)
    scale = torch.as_tensor(SCALE, device=DEV).double()
    if not training:
        pred = x.clone()
        pred[..., :6] += scale * out[..., :6]
        return {"pred": pred.reshape(-1), "out": out.reshape(-1)}
    mask = x[..., 6:7]
    e = (x[..., :6] + scale * out[..., :6] - tgt[..., :6]) / scale
    m = mask[..., 0]
    mass = (m * (x[..., 0] + scale[0] * out[..., 0] - tgt[..., 0])).sum() / (m * tgt[..., 0]).sum()
    loss = (mask * e * e).sum() / (6 * mask.sum()) + 100.0 * mass * mass
    loss.backward()
    g = torch.zeros(net.nparam, dtype=torch.float64, device=DEV)
    for name, (o, nw, ob, nb) in parts.items():
        g[o:o + nw], g[ob:ob + nb] = weights[name][0].grad.reshape(-1), weights[name][1].grad
    # the updated weights follow the sign of gradients near zero: no value of their own
    return {"loss": np.array([float(loss.detach()), float(mass.detach())]), "g": g, "p": None,
            "out": out.detach().reshape(-1)}


def exact_circuit(case, seed):
    """The potentials by a dense solve over the beads that reach an electrode."""
    pos, x_src, x_snk = circuit(case, seed)
    pos = torch.from_numpy(pos).to(DEV)
    d = pos[:, None] - pos[None]
    r2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
    join = (r2 > 0) & (r2 < 5.25 * 5.25)
    G = torch.where(join, 1 / torch.where(join, r2, torch.ones_like(r2)).sqrt(), torch.zeros_like(r2))
    src, snk = pos[:, 0] < x_src, pos[:, 0] > x_snk
    reach = src | snk
    while True:
        more = reach | (join & reach[None]).any(1)
        if bool((more == reach).all()):
            break
        reach = more
    free = reach & ~src & ~snk
    V = src.double()
    if bool(free.any()):
        A = torch.diag(G.sum(1)) - G
        b = (G * V[None]).sum(1)
        V[free] = torch.from_numpy(np.linalg.solve(A[free][:, free].cpu().numpy(), b[free].cpu().numpy())).to(DEV)
    cur = G * (V[:, None] - V[None])
    total = float(cur[src][:, ~src].sum())
    gap = x_snk - x_src
    return {"V": V, "I": 0.5 * cur.abs().sum(1), "I_tot": total, "I_ref": 1 / gap, "kappa": total * gap,
            "edges": None, "n_source": None, "n_sink": None, "max_degree": None}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("sphere", "cap", "cg"):
        rho, mat, p = fluid_inputs(case, seed)
        rho, mat = torch.from_numpy(rho).to(DEV), torch.from_numpy(mat).to(DEV)
        fluid = mat == 0
        f = torch.as_tensor(Wt, device=DEV, dtype=torch.float64)[None, :, None, None, None] * (rho * fluid)[:, None]
        for _ in range(case["steps"]):
            if kind == "cg":
                f = colour_gradient(f, mat, fluid, p.cg_sigma, p.cg_beta, p.cg_theta)
            else:
                f = shan_chen(f, mat, fluid, p.G, p.rho_top)
        return {"rho": f.sum(1), "f": f}
    if kind in ("predict", "train"):
        return exact_network(case, seed, kind == "train")
    if kind == "conv":
        x1, x2, w, b, dy = conv_inputs(case, seed)
        x = up64(x1.double()) if case["up"] else x1.double()
        x = torch.cat([x, x2.double()], dim=-1) if x2 is not None else x
        x, w, b = (t.double().requires_grad_(True) for t in (x, w, b))
        y = torch.relu(conv64(x, w, b))
        y.backward(dy.double())
        return {"y": y.detach(), "dx": x.grad, "dw": w.grad, "db": b.grad}
    if kind == "network":
        return exact_circuit(case, seed)
    # the coupled runs: the rods' and beads' passes take a 64-bit program of
    # their own far over 20 seconds at these sizes; the analysis is counts
    # and FP64 reductions
    return None
