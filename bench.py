"""Throughput of the coupled Shan-Chen D3Q19 step on one MI355X.

Workload (default): the elongated sessile cap on the 256 x 128 x 64 lattice
(footprint 150 x 36, height 24, stripe 160 x 40, reservoir plane on top),
FP32 populations.  One step = one pass of the hot path over the lattice.
Inputs are resident in HBM before the timed region starts.

Prints ONE JSON line with the metric (MLUPS over fluid nodes), a roofline
object for the two kernels of a fluid step inside a call of many (the bytes
that they cannot do without / the fluid step's time, from HIP events on the
launch stream) and the FP64 oracle timed on the host cores on a bounded sample
of the same workload.
"""
from __future__ import annotations

import os

# the oracle's baseline is single-threaded by construction; pin BLAS pools too
for _v in ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS", "MKL_NUM_THREADS"):
    os.environ.setdefault(_v, "1")

import argparse  # noqa: E402
import json  # noqa: E402
import sys  # noqa: E402
import time  # noqa: E402

import numpy as np  # noqa: E402

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X published HBM3E bandwidth
BYTES_PER_ELEM = {"f64": 8, "f32": 4, "f16dev": 2, "bf16dev": 2}
METRIC = "MLUPS + % HBM roofline: plain vs FP16-storage vs batched; surrogate speedup"


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def algorithmic_bytes_per_lu(prec):
    # every population of both components read once and written once
    return 2 * 19 * 2 * BYTES_PER_ELEM[prec]


def step_bytes_per_lu(prec, rho_ref=0.0):
    # a fluid step inside a call: the stream pass and the collide pass, which
    # pass on psi_k and j (with a storage reference also rho_k - rho_ref) in
    # compute precision.  FP32 and FP64 steps go from moments to moments (per
    # component rho, u and the rest population); 16-bit ones from populations
    # to populations
    c = 8 if prec == "f64" else 4
    state = 10 * c if prec in ("f32", "f64") else 2 * 19 * BYTES_PER_ELEM[prec]
    return 2 * state + 2 * (5 + (2 if rho_ref else 0)) * c


# 16-bit storage forms: (storage, reference density) -- rho_ref = 0 stores
# f_i itself, rho_ref = 1 stores the deviation f_i - w_i from the lattice weights
FORMS16 = {"f16": ("f16dev", 0.0), "bf16": ("bf16dev", 0.0), "f16dev": ("f16dev", 1.0), "bf16dev": ("bf16dev", 1.0)}


def storage_error_report(steps=10000):
    """Error of each 16-bit storage form against the FP64 oracle on the
    static-droplet workload (32^3 periodic, R = 8) after `steps` steps: the
    oracle's fields and the random-rounding model's errors are the stored
    expected values of tests/golden/make_config3_oracle.py."""
    import torch

    from paper_2607_06794_amd.sim import Lattice
    from tests import cases
    from tests.golden import errors as G

    gold = np.load(G.CONFIG3_ORACLE)
    model = json.load(open(G.CONFIG3_MODEL))["forms"]
    c = cases.sphere_case()
    out = {}
    for name, (prec, ref) in FORMS16.items():
        lat = Lattice(cases.lattice_params(c, prec, rho_ref=(ref, ref), rounding="stochastic"), c["rho"], c["mat"])
        m0 = lat.observables(allow_unstable=True)["mass"]
        lat.step(steps)
        obs = lat.observables(allow_unstable=True)
        rho, f = lat.export()
        lat.close()
        torch.cuda.synchronize()
        u = G.velocity(rho, f)
        rho_o, u_o = gold["rho"].astype(np.float64), gold["u"].astype(np.float64)
        err = G.field_errors(rho, u, rho_o, u_o, obs["mass"], gold["mass"])
        err["mass_rel"] = [float(abs(obs["mass"][k] - m0[k]) / m0[k]) for k in range(2)]
        err["aligned"] = G.aligned_errors(rho, u, rho_o, u_o)
        fmt = "f16" if prec == "f16dev" else "bf16"
        runs = model[f"{fmt}|rho_ref={ref:g}"]
        out[name] = {"steps": steps, "rounding": "stochastic", "status": int(obs["status"]), "error": err,
                     "model_aligned_rho_A_max": max(r["aligned"]["rho_A"]["max"] for r in runs),
                     "model_drift_max": max(float(np.linalg.norm(r["aligned"]["displacement"])) for r in runs),
                     "mass_walk_sigma": G.rounding_walk(rho_o, ref, fmt, steps)}
        log(f"[bench] storage {name}: rho_A max {err['rho_A']['max']:.3e} (aligned {err['aligned']['rho_A']['max']:.3e},"
            f" model {out[name]['model_aligned_rho_A_max']:.3e}), drift "
            f"{np.linalg.norm(err['aligned']['displacement']):.3f} (model {out[name]['model_drift_max']:.3f})")
    return out


def rod_params(lp, length=24.0):
    lp.rod_length, lp.rod_radius, lp.rod_rho = length, 2.0, 1.0
    lp.eps_att, lp.eps_rep, lp.rod_d0, lp.rod_rcut = 1e-4, 0.03, 5.0, 7.5
    lp.eps_wall, lp.rod_d0_wall, lp.n_sub, lp.wall_z = 0.03, 3.0, 5, 0.5
    return lp


def time_step(case, prec, steps, warmup, tile, rods=None, segment=0, rho_ref=(0.0, 0.0), rounding="nearest"):
    """Time `steps` coupled steps (fluid step + rod update).

    With rods, the steps run in segments of at most `segment` steps, each
    from a freshly initialised lattice (untimed set-up and `warmup` steps
    before the first segment only): rods placed anywhere in the fluid (the
    stress placement) cross the liquid-vapour interface and the coupled state
    degrades after a few hundred steps, and timing a degraded state would time
    less rod work.  A segment is one call of that many steps.  Returns (ms per
    whole step inside a call, ms per fluid step in a call of its own, fluid
    nodes, observables of the last segment, segments).  The second
    comes from a pair of HIP events around each of up to 100 calls of one step
    on a fresh lattice, after the timed segments: such a call goes from
    populations to populations, while FP32 and FP64 steps inside a call pass on
    moments.
    """
    import torch

    from paper_2607_06794_amd.sim import Lattice
    from tests import cases

    lp = rod_params(cases.lattice_params(case, prec, rho_ref=rho_ref, rounding=rounding, **tile))
    seg = steps if (rods is None or segment <= 0) else min(segment, steps)
    total_ms = 0.0
    done = nseg = 0
    n_fluid = 0
    obs = None
    worst = 0
    while done < steps:
        lat = Lattice(lp, case["rho"], case["mat"], rods=rods)
        if nseg == 0:
            n_fluid = int(lat.observables()["fluid_nodes"])
            lat.coupled_step(warmup)
        n = min(seg, steps - done)
        torch.cuda.synchronize()
        stream = torch.cuda.current_stream()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        lat.coupled_step(n)
        e1.record(stream)
        torch.cuda.synchronize()
        total_ms += e0.elapsed_time(e1)
        obs = lat.observables(allow_unstable=True)
        worst |= int(obs["status"])
        lat.close()
        done += n
        nseg += 1
    obs["status"] = worst
    single = min(steps, 100)
    lat = Lattice(lp, case["rho"], case["mat"], rods=rods)
    lat.coupled_step(min(warmup, 10))
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(single)]
    for a, b in ev:
        a.record(stream)
        lat.step(1)
        b.record(stream)
        lat.rods_step()
    torch.cuda.synchronize()
    single_ms = sum(a.elapsed_time(b) for a, b in ev)
    lat.close()
    return total_ms / steps, single_ms / single, n_fluid, obs, nseg


def batched_form(steps, warmup, n_lattices=64):
    """Many-droplet sweep: every lattice stepped alone, one after another, against
    the batched step (shared launches for each pass) with and
    without the HIP graph, fluid-only and coupled (with rods).  Each coupled
    variant starts from freshly initialised lattices (rods placed anywhere in
    the fluid degrade the state within a few hundred steps)."""
    import torch

    from paper_2607_06794_amd import inputs
    from paper_2607_06794_amd.sim import Batch, Lattice
    from tests import cases

    specs = list(inputs.sweep_droplets(n_lattices))

    def make():
        lats = []
        for d in specs:
            c = dict(shape=d["shape"], periodic=(True, True, False), G=3.6, tau=(1.0, 1.0), evaporation=True,
                     body_force=(0.0, 0.0, 0.0))
            lp = rod_params(cases.lattice_params(c, "f32"), length=d["rod_length"])
            lp.eps_att = d["eps_att"]
            lats.append(Lattice(lp, d["rho"], d["mat"], rods=d["rods"]))
        torch.cuda.synchronize()
        return lats

    stream = torch.cuda.current_stream()

    def timed(fn, n):
        fn(warmup)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        fn(n)
        e1.record(stream)
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / n

    def solo(lats, rods):
        def run(n):
            for _ in range(n):
                for lat in lats:
                    lat.step(1)
                    if rods:
                        lat.rods_step()
        return run

    n_fluid = sum(int((d["mat"] == 0).sum()) for d in specs)
    out = {"lattices": len(specs), "fluid_nodes": n_fluid,
           "rods": int(sum(0 if d["rods"] is None else len(d["rods"]) for d in specs))}
    for rods in (False, True):
        res = {}
        for variant in ("solo", "batched", "graph"):
            lats = make()
            if variant == "solo":
                ms = timed(solo(lats, rods), steps)
            else:
                batch = Batch(lats, stream=stream)
                ms = timed(lambda n: batch.step(n, rods=rods, graph=(variant == "graph")), steps)
                batch.close()
            st = 0
            for lat in lats:
                st |= int(lat.observables(allow_unstable=True)["status"])
                lat.close()
            res[variant] = (ms, st)
        key = "coupled" if rods else "fluid"
        out[key] = {f"ms_per_step_{v}": res[v][0] for v in res}
        out[key].update({f"mlups_{v}": n_fluid / (res[v][0] * 1e-3) / 1e6 for v in res})
        out[key]["speedup_vs_solo"] = res["solo"][0] / min(res["batched"][0], res["graph"][0])
        out[key]["status"] = {v: res[v][1] for v in res}
        log(f"[bench] batched {key}: solo {res['solo'][0]:.2f} ms, batched {res['batched'][0]:.2f} ms, "
            f"graph {res['graph'][0]:.2f} ms per step")
    shapes = ["{2}x{1}x{0}".format(*d["shape"]) for d in specs]
    out["grid_classes"] = {k: shapes.count(k) for k in sorted(set(shapes))}
    return out


def surrogate_form(n_droplets=64, n_snap=8, interval=500, epochs=2, warm=200, K=50, jump_after=3, lam=100.0,
                   n_ens=12, drift=0.5, log_fn=None):
    """Learned surrogate: LBM trajectories of the droplet sweep (physically
    placed rods) restricted to the 128 x 64 x 32 canvas every `interval` steps;
    the U-Net is trained with the library's kernels on the first 7/8 of the
    droplets and evaluated on the rest against persistence and linear
    extrapolation; then one interval of every test droplet is timed both
    ways, from step warm + jump_after x interval: `interval` LBM steps
    against SU.advance (state snapshot for the fallback, restrict, network,
    rod jump, lift, K re-equilibration steps) with its 0.5 % mass rule
    applied.  The speed-up is quoted over the jumps
    that pass the rule, with their count; the effective speed-up includes
    the fallbacks."""
    import torch

    from paper_2607_06794_amd import inputs
    from paper_2607_06794_amd import surrogate as SU
    from paper_2607_06794_amd.sim import Batch, Lattice
    from tests import cases

    D, H, W = 32, 64, 128
    specs = list(inputs.sweep_droplets(n_droplets, placement="physical"))

    def make(d):
        c = dict(shape=d["shape"], periodic=(True, True, False), G=3.6, tau=(1.0, 1.0), evaporation=True,
                 body_force=(0.0, 0.0, 0.0))
        lp = rod_params(cases.lattice_params(c, "f32"), length=d["rod_length"])
        lp.eps_att = d["eps_att"]
        return Lattice(lp, d["rho"], d["mat"], rods=d["rods"] if d["rods"] is not None and len(d["rods"]) else None)

    def expected_loss(m_pp, m_prev, m_now):
        """rho_A mass the lattice is expected to lose over the next interval
        from its masses at the starts of the two intervals before and now:
        in the drying phase the loss per interval falls by a roughly
        constant ratio from one interval to the next (on the sweep's test
        droplets this halves the error of taking the last loss again, to
        about 0.13 % of the mass), so the last loss times that ratio while
        it falls, else the last loss."""
        l0, l1 = m_pp - m_prev, m_prev - m_now
        return l1 * (l1 / l0) if 0.0 < l1 < l0 else l1

    def rods_centres(lat):
        """Rod centres (CUDA FP64 [n, 3]) for a jump that continues each
        rod's displacement since now; None when the jump holds the rods."""
        if drift < 0 or not lat.n_rods:
            return None
        return torch.from_numpy(np.ascontiguousarray(lat.rods()[:, :3])).to(lat.device)

    lats = [make(d) for d in specs]
    batch = Batch(lats)
    t0 = time.perf_counter()
    xf, xb, healthy = SU.rollout_snapshots(batch, lats, n_snap, interval, D, H, W, warm=warm, log=log_fn)
    t_gen = time.perf_counter() - t0
    batch.close()
    lat_status = []
    for lat in lats:
        lat_status.append(int(lat.observables(allow_unstable=True)["status"]))
        lat.close()
    # pairs only from lattices whose status word is still clear at the later
    # snapshot: states on the way to an instability are not training data
    finite = torch.isfinite(xf.view(len(specs), n_snap, -1)).all(dim=2).cpu().numpy() & healthy
    ntrain = len(specs) * 7 // 8
    train = [(xf[i, s], xb[i, s], xf[i, s + 1]) for i in range(ntrain) for s in range(n_snap - 1)
             if finite[i, s] and finite[i, s + 1]]
    test = [(xf[i, s], xb[i, s], xf[i, s + 1]) for i in range(ntrain, len(specs)) for s in range(1, n_snap - 1)
            if finite[i, s] and finite[i, s + 1] and finite[i, s - 1]]
    prev = [xf[i, s - 1] for i in range(ntrain, len(specs)) for s in range(1, n_snap - 1)
            if finite[i, s] and finite[i, s + 1] and finite[i, s - 1]]
    net = SU.UNet(D, H, W).init(0)
    t0 = time.perf_counter()
    hist = SU.fit(net, train, epochs=epochs, batch=4, lr=3e-4, lam=lam, log=log_fn)
    torch.cuda.synchronize()
    t_train = time.perf_counter() - t0
    ev = SU.evaluate(net, test, lam=lam, prev=prev)
    # forward throughput of the network (matrix-core work)
    flops = sum(2.0 * 27 * (c1 + c2) * co * net.P[lvl] for _, c1, c2, co, _, lvl in net.layers)
    stream = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    net.forward(test[0][1])
    e0.record(stream)
    for _ in range(10):
        net.forward(test[0][1])
    e1.record(stream)
    torch.cuda.synchronize()
    ms_fwd = e0.elapsed_time(e1) / 10
    # one interval of every test droplet, both ways: `interval` LBM steps
    # against SU.advance with its fallback rule applied (a jump whose rho_A
    # mass misses M_t - rate * interval by more than 0.5 % restores the
    # snapshot and runs the plain interval, and that time counts too).  The
    # speed-up is quoted over the jumps that pass the rule; the effective one
    # includes the fallbacks.
    # The jumps start at t0 = warm + jump_after x interval, in the slow drying
    # phase: over the first intervals of a fresh cap the mass loss rate still
    # halves from one interval to the next, and M_t - rate x interval (rate
    # from the interval before) misses the method's own mass at t0 + interval
    # by 3-8 % at t0 = warm, against 0.2-0.4 % from t0 = warm + 3 intervals.
    # The rate comes from the rho_A mass the lattice lost over the two
    # intervals before t0, from every cause (reservoir and rods):
    # expected_loss.  Each trial also
    # reports the rule's error on the method's own trajectory (its
    # resolution) and the jump's mass error against the method.
    t0 = warm + jump_after * interval
    trials = []
    keep = None
    ens_pick = None
    for idx in range(ntrain, len(specs)):
        lat_a, lat_b = make(specs[idx]), make(specs[idx])
        for lat in (lat_a, lat_b):
            lat.coupled_step(t0 - 2 * interval)
        m_pp = float(lat_b.observables(allow_unstable=True)["mass"][0])
        for lat in (lat_a, lat_b):
            lat.coupled_step(interval)
        m_prev = float(lat_b.observables(allow_unstable=True)["mass"][0])
        x_prev = rods_centres(lat_b)
        for lat in (lat_a, lat_b):
            lat.coupled_step(interval)
        ob = lat_b.observables(allow_unstable=True)
        nodes = int(np.prod(specs[idx]["shape"]))
        if int(ob["status"]) & 3:  # NaN or a non-positive density before the jump: no trial
            trials.append({"droplet": idx, "nodes": nodes, "skipped": f"status {int(ob['status'])} at step {t0}"})
            lat_a.close()
            lat_b.close()
            continue
        m_now = float(ob["mass"][0])
        rate = expected_loss(m_pp, m_prev, m_now) / interval
        torch.cuda.synchronize()
        e0.record(stream)
        lat_a.coupled_step(interval)
        e1.record(stream)
        torch.cuda.synchronize()
        ms_lbm = e0.elapsed_time(e1)
        e0.record(stream)
        adv = SU.advance(lat_b, net, D, H, W, interval=interval, K=K, rate=rate, threshold=0.005, rods_prev=x_prev,
                         drift=drift)
        e1.record(stream)
        torch.cuda.synchronize()
        ms_sur = e0.elapsed_time(e1)
        oa = lat_a.observables(allow_unstable=True)
        m_lbm = float(oa["mass"][0])
        trials.append({"droplet": idx, "nodes": nodes, "ms_lbm": ms_lbm, "ms_advance": ms_sur,
                       "passed": bool(adv["surrogate"]), "jump_mass_error": float(adv["mass_error"]),
                       "rule_error_of_lbm": abs(m_lbm - (m_now - rate * interval)) / m_now,
                       "jump_mass_error_vs_lbm": abs(float(adv["mass"]) - m_lbm) / m_lbm,
                       "lbm_status": int(oa["status"])})
        # accuracy figures on the largest test droplet with rods whose jump
        # passed (else the largest with rods, else the largest); the ensemble
        # below takes the largest tried droplet with rods whatever its jump did
        has_rods = lat_b.n_rods > 0
        if has_rods and (ens_pick is None or nodes > ens_pick[1]):
            ens_pick = (idx, nodes)
        key = (bool(adv["surrogate"]) and has_rods, has_rods, nodes)
        if keep is None or key > keep[7]:
            if keep is not None:
                keep[0].close()
                keep[1].close()
            keep = [lat_a, lat_b, idx, rate, bool(adv["surrogate"]), nodes, adv, key]
        else:
            lat_a.close()
            lat_b.close()
    if keep is None:  # every test droplet failed before the jump
        return {"canvas": [W, H, D], "droplets": len(specs), "train_pairs": len(train), "test_pairs": len(test),
                "test_loss": ev, "jump_at_step": t0, "jumps_tried": 0, "jumps_passed": 0, "jumps": trials}
    lat_a, lat_b, idx, rate, _, _, adv, _ = keep
    tried = [t for t in trials if "skipped" not in t]
    passed = [t for t in tried if t["passed"]]
    ms_lbm = float(np.mean([t["ms_lbm"] for t in passed])) if passed else None
    ms_sur = float(np.mean([t["ms_advance"] for t in passed])) if passed else None
    eff = sum(t["ms_lbm"] for t in tried) / sum(t["ms_advance"] for t in tried)
    nzl, nyl, nxl = specs[idx]["shape"]
    dspec = (16, 4, (nxl - 1) / 2, (nyl - 1) / 2, float(nxl), nyl / 2.0)

    def compare(ref, other):
        """rho_A mass, deposit map, g^b (x) (Eq. 14), rod positions and
        contact graph of `other` against `ref`."""
        ma = ref.observables(allow_unstable=True)
        mb = other.observables(allow_unstable=True)
        # deposit: L1 distance of the z-projected rod-fraction maps of the
        # two states on the canvas, over the reference map's total
        ca, _ = SU.restrict(ref, D, H, W)
        cb, _ = SU.restrict(other, D, H, W)
        rmap_a = ca.view(D, H, W, 8)[..., 5].sum(dim=0).cpu().numpy()
        rmap_b = cb.view(D, H, W, 8)[..., 5].sum(dim=0).cpu().numpy()
        da, db = ref.deposit(*dspec), other.deposit(*dspec)
        ra, rb = ref.rods(), other.rods()
        dx_r = rb[:, :3] - ra[:, :3]
        for ax, n in ((0, nxl), (1, nyl)):
            dx_r[:, ax] -= n * np.round(dx_r[:, ax] / n)
        return {"mass": float(abs(mb["mass"][0] - ma["mass"][0]) / ma["mass"][0]),
                "deposit": float(np.abs(rmap_a - rmap_b).sum() / max(rmap_a.sum(), 1e-30)) if rmap_a.sum() > 0 else 0.0,
                "g_x": float(np.abs(da["g_x"] - db["g_x"]).mean()),
                "rods": float(np.sqrt((dx_r ** 2).sum(axis=1)).mean()) if len(ra) else 0.0,
                "edges": [int(da["edges"]), int(da["largest"]), int(db["edges"]), int(db["largest"])],
                "status": int(mb["status"])}

    acc = compare(lat_a, lat_b)
    # the method against itself: the kept droplet's state at t0 with every
    # stored population scaled by 1 + 1e-6 u (u uniform in [-1, 1], seeded),
    # run over the same interval; the same figures then give the resolution
    # that one trajectory allows for each of them (the coupled dynamics
    # amplifies such differences)
    # (a twin run to t0: the steps are deterministic, and a snapshot goes
    # back only into the lattice it came from)
    lat_c = make(specs[idx])
    lat_c.coupled_step(t0)
    snap_c = lat_c.snapshot()
    f32 = snap_c[0].view(torch.float32)
    gen = torch.Generator(device=f32.device).manual_seed(7)
    f32.mul_(1.0 + 1e-6 * (2.0 * torch.rand(f32.shape, generator=gen, device=f32.device) - 1.0))
    lat_c.restore(snap_c)
    lat_c.coupled_step(interval)
    own = compare(lat_a, lat_c)
    lat_c.close()

    # The deposit density as the paper measures it (the g^b profile of
    # Eq. 14 averaged over independent runs and their mirror images): n_ens
    # runs of the accuracy droplet's configuration (the cap's noise and the
    # rod placement drawn anew), each carried from t0 over one interval by
    # the method, by a jump (taken whatever the mass rule says, so that this
    # measures the network; the rule's verdicts are counted), and by the
    # method from populations scaled by 1 + 1e-6 u at t0 (the resolution).
    ens = None
    if n_ens > 0 and ens_pick is not None:
        eidx = ens_pick[0]
        enz, eny, enx = specs[eidx]["shape"]
        edspec = (16, 4, (enx - 1) / 2, (eny - 1) / 2, float(enx), eny / 2.0)
        from paper_2607_06794_amd.sim import deposit_ensemble

        lbm_runs, sur_runs, own_runs, per_sur, per_own, runs_info = [], [], [], [], [], []
        passes = 0
        for run in range(n_ens):
            d = next(inputs.sweep_droplets(eidx + 1, placement="physical", first=eidx, run=run))
            if d["rods"] is None or len(d["rods"]) == 0:
                runs_info.append({"run": run, "skipped": "no rod fits"})
                continue
            la, lb, lc = make(d), make(d), make(d)
            for lat in (la, lb, lc):
                lat.coupled_step(t0 - 2 * interval)
            m_pp = float(lb.observables(allow_unstable=True)["mass"][0])
            for lat in (la, lb, lc):
                lat.coupled_step(interval)
            m_prev = float(lb.observables(allow_unstable=True)["mass"][0])
            x_prev_r = rods_centres(lb)
            for lat in (la, lb, lc):
                lat.coupled_step(interval)
            ob = lb.observables(allow_unstable=True)
            if int(ob["status"]) & 3:
                runs_info.append({"run": run, "skipped": f"status {int(ob['status'])} at step {t0}"})
                for lat in (la, lb, lc):
                    lat.close()
                continue
            rate_r = expected_loss(m_pp, m_prev, float(ob["mass"][0])) / interval
            snap = lc.snapshot()
            f32 = snap[0].view(torch.float32)
            gen = torch.Generator(device=f32.device).manual_seed(100 + run)
            f32.mul_(1.0 + 1e-6 * (2.0 * torch.rand(f32.shape, generator=gen, device=f32.device) - 1.0))
            lc.restore(snap)
            del snap, f32
            la.coupled_step(interval)
            lc.coupled_step(interval)
            st_ac = [int(lat.observables(allow_unstable=True)["status"]) for lat in (la, lc)]
            if (st_ac[0] | st_ac[1]) & 3:  # the method itself failed over the interval: no member
                runs_info.append({"run": run, "skipped": f"method status {st_ac} after the interval"})
                for lat in (la, lb, lc):
                    lat.close()
                continue
            r = SU.advance(lb, net, D, H, W, interval=interval, K=K, rate=rate_r, threshold=1.0, rods_prev=x_prev_r,
                           drift=drift)
            passes += int(r["mass_error"] <= 0.005)
            ga, gb, gc = (lat.deposit(*edspec)["g_x"] for lat in (la, lb, lc))
            per_sur.append(float(np.abs(ga - gb).mean()))
            per_own.append(float(np.abs(ga - gc).mean()))
            runs_info.append({"run": run, "rods": int(la.n_rods), "g_x_error": per_sur[-1], "g_x_error_own": per_own[-1],
                              "status": [int(lat.observables(allow_unstable=True)["status"]) for lat in (la, lb, lc)]})
            lbm_runs.append(la)
            sur_runs.append(lb)
            own_runs.append(lc)
        if lbm_runs:
            ea, eb, ec = (deposit_ensemble(runs, *edspec, mirror=True)["g_x"]
                          for runs in (lbm_runs, sur_runs, own_runs))
            ens = {"droplet": eidx, "runs": len(lbm_runs), "runs_tried": n_ens, "mirror_images": True, "from_step": t0,
                   "g_x_error": float(np.abs(ea - eb).mean()), "g_x_error_own": float(np.abs(ea - ec).mean()),
                   "per_run_g_x_error": float(np.mean(per_sur)), "per_run_g_x_error_own": float(np.mean(per_own)),
                   "jumps_within_rule": passes, "g_x_lbm": ea.tolist(), "g_x_surrogate": eb.tolist(),
                   "g_x_own": ec.tolist(), "per_run": runs_info}
        for lat in lbm_runs + sur_runs + own_runs:
            lat.close()
        if log_fn and ens:
            log_fn(f"[surrogate] ensemble of {ens['runs']} runs with mirror images: g_x error "
                   f"{ens['g_x_error']:.4f} (the method against itself {ens['g_x_error_own']:.4f}; one run "
                   f"{ens['per_run_g_x_error']:.4f} / {ens['per_run_g_x_error_own']:.4f}), "
                   f"{passes} of {ens['runs']} jumps within the rule")
    mass_err, dep_err, g_err, rod_err = acc["mass"], acc["deposit"], acc["g_x"], acc["rods"]
    ra = lat_a.rods()
    status_b = acc["status"]
    lat_a.close()
    lat_b.close()
    # end-of-rollout status words by what they flag: NaN (bit 1), a
    # non-positive density without NaN (bit 2), a rod limit only (bits 8, 16,
    # 32), the speed bit alone (4: also set by the near-empty layer under the
    # reservoir), or nothing
    status_kinds = {
        "clear": sum(1 for st in lat_status if st & ~64 == 0),
        "speed_only": sum(1 for st in lat_status if st & ~64 == 4),
        "far_refill_notice": sum(1 for st in lat_status if st & 64),
        "rod_limit": sum(1 for st in lat_status if st & 56 and not st & 3),
        "nonpositive_density": sum(1 for st in lat_status if st & 2 and not st & 1),
        "nan": sum(1 for st in lat_status if st & 1),
    }
    n_unstable = int(sum(1 for st in lat_status if st & ~(4 | 64)))  # 64: far-refill notice
    out = {
        "canvas": [W, H, D], "droplets": len(specs), "train_pairs": len(train), "test_pairs": len(test),
        "interval_steps": interval, "reequilibration_steps": K, "params": int(net.nparam),
        "data_generation_s": t_gen, "train_s": t_train, "epochs": epochs, "mass_loss_weight": lam, "rod_drift": drift,
        "train_loss": hist,
        "test_loss": ev, "gain_over_persistence": ev["persistence"] / max(ev["net"], 1e-30),
        "fwd_ms": ms_fwd, "fwd_tflops": flops / (ms_fwd * 1e-3) / 1e12, "fwd_gflop_per_sample": flops / 1e9,
        "jump_at_step": t0, "jumps_tried": len(tried), "jumps_passed": len(passed), "jumps": trials,
        "ms_lbm_interval": ms_lbm, "ms_surrogate_interval": ms_sur,
        "speedup": (ms_lbm / ms_sur) if passed else None,
        "speedup_note": "mean over the test droplets whose jump passed the 0.5 % mass rule",
        "speedup_with_fallbacks": eff,
        "accuracy_droplet": idx, "accuracy_jump_passed": bool(adv["surrogate"]),
        "mass_error_vs_lbm": mass_err, "deposit_error_vs_lbm": dep_err, "g_x_error_vs_lbm": g_err,
        "rod_position_error": rod_err, "rods": int(len(ra)),
        "contacts": {"lbm": acc["edges"][:2], "surrogate": acc["edges"][2:]},
        "lbm_self_sensitivity": {"perturbation": "populations x (1 + 1e-6 u) at the jump's start", **own},
        "deposit_ensemble": ens,
        "fallback_threshold": 0.005, "jump_mass_error": float(adv["mass_error"]),
        "reservoir_rate_per_step": float(rate),
        "status_after_jump": status_b,
        "rollout_unstable_droplets": n_unstable, "rollout_status": status_kinds, "pairs_dropped_unhealthy": int(
            (len(specs) * 7 // 8) * (n_snap - 1) - len(train) + (len(specs) - len(specs) * 7 // 8) * (n_snap - 2) - len(test)),
    }
    if log_fn:
        sp = "n/a" if out["speedup"] is None else f"x{out['speedup']:.2f}"
        log_fn(f"[surrogate] gain over persistence x{out['gain_over_persistence']:.2f}, jumps passed "
               f"{len(passed)}/{len(tried)}, speedup {sp} (x{eff:.2f} with fallbacks), "
               f"mass error {mass_err:.2e}, deposit error {dep_err:.3f}, g_x error {g_err:.3f}, rod error {rod_err:.2f}, "
               f"forward {ms_fwd:.2f} ms ({out['fwd_tflops']:.1f} TFLOP/s), rollouts at the end {status_kinds}")
    return out


def _finite(v):
    """The record with every non-finite float as null (strict JSON)."""
    if isinstance(v, dict):
        return {k: _finite(x) for k, x in v.items()}
    if isinstance(v, (list, tuple)):
        return [_finite(x) for x in v]
    if isinstance(v, (float, np.floating)):
        return float(v) if np.isfinite(v) else None
    if isinstance(v, np.integer):
        return int(v)
    if isinstance(v, np.bool_):
        return bool(v)
    return v


def unet_form(reps=20):
    """U-Net alone on the 128 x 64 x 32 canvas of the 256 x 128 x 64 cap at
    t = 0: forward and forward + backward, timed with events on the
    network's stream.  One JSON line; used to profile the convolutions."""
    import torch

    from paper_2607_06794_amd import surrogate as SU
    from paper_2607_06794_amd.sim import Lattice
    from tests import cases

    D, H, W = 32, 64, 128
    c = cases.cap_case()
    lat = Lattice(cases.lattice_params(c, "f32"), c["rho"], c["mat"])
    lat.step(50)
    xf, _ = SU.restrict(lat, D, H, W)
    lat.close()
    net = SU.UNet(D, H, W).init(0)
    tgt = xf.clone()
    gout = torch.zeros(net.P[0] * SU.COUT, dtype=torch.float32, device=xf.device)
    flops = sum(2.0 * 27 * (c1 + c2) * co * net.P[lvl] for _, c1, c2, co, _, lvl in net.layers)
    stream = net.stream
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(3):
        net.forward(net.prepare(xf))
    e0.record(stream)
    for _ in range(reps):
        net.forward(net.prepare(xf))
    e1.record(stream)
    torch.cuda.synchronize()
    ms_f = e0.elapsed_time(e1) / reps
    net.forward(net.prepare(xf))
    net.loss(xf, tgt, 1.0, grad=gout)
    e0.record(stream)
    for _ in range(reps):
        net.zero_grad()
        net.backward(gout)
    e1.record(stream)
    torch.cuda.synchronize()
    ms_b = e0.elapsed_time(e1) / reps
    return {"metric": "U-Net forward and backward", "canvas": [W, H, D], "params": int(net.nparam),
            "gflop_forward": flops / 1e9, "ms_forward": ms_f, "ms_backward": ms_b,
            "tflops_forward": flops / (ms_f * 1e-3) / 1e12, "tflops_backward": 2 * flops / (ms_b * 1e-3) / 1e12,
            "peak_tflops_bf16": 2500.0, "dtype": "bf16 (fp32 accumulate)", "data": "synthetic"}


def copy_probe(mib, reps=5):
    """A plain device copy of `mib` MiB (torch copy_, source written first):
    the known byte count against which the FETCH_SIZE and WRITE_SIZE
    counters are scaled, and the copy rate (HIP events around the `reps`
    copies on the current stream; bytes read plus written)."""
    import torch

    n = mib * (1 << 20) // 4
    src = torch.ones(n, dtype=torch.float32, device="cuda:0")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    for _ in range(reps):
        dst.copy_(src)
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / reps
    return {"metric": "copy probe", "bytes_read": n * 4, "bytes_written": n * 4, "reps": reps + 1,
            "us_per_copy": ms * 1e3, "gbs_read_plus_written": 2 * n * 4 / (ms * 1e-3) / 1e9}


def traffic_record(prec, n_fluid, ms_fluid, rods=False):
    """Measured HBM traffic of a fluid step inside a call from the committed
    counter record (FETCH_SIZE and WRITE_SIZE per launch of its two kernels,
    each scaled by what the counter reads for a plain copy of known size), or
    None when the record does not describe this kernel source, precision and
    lattice."""
    import hashlib

    path = os.path.join(ROOT, "profiles", "sc_step_traffic.json")
    try:
        with open(path) as fh:
            rec = json.load(fh)
        with open(os.path.join(ROOT, "paper_2607_06794_amd", "csrc", "sc_step.hip"), "rb") as fh:
            sha = hashlib.sha256(fh.read()).hexdigest()
    except (OSError, ValueError):
        return None
    if rec.get("sc_step_sha256") != sha or rec.get("prec") != prec or rec.get("fluid_nodes") != n_fluid \
            or bool(rec.get("rods", False)) != bool(rods):
        return None
    b = sum(1024.0 * (k["fetch_kib"] * rec["fetch_scale"] + k["write_kib"] * rec["write_scale"])
            for k in rec["kernels"].values())
    return {"bytes_per_step": b, "gbs": b / (ms_fluid * 1e-3) / 1e9,
            "vs_needed": b / (step_bytes_per_lu(prec) * n_fluid)}


def network_form(case, reps=5, n_rods=300, seed=5000):
    """The deposit's resistor network (Eqs. 15-18) on a dried deposit: n_rods
    rods of the benchmark's shape lying crossed on the substrate of the
    256 x 128 x 64 cap (inputs.deposit_rods: centres uniform in x 40-216,
    y 4-124 at z 3.5, directions at a uniform angle), as beads every 2 nodes
    along each axis (lb_rod_beads), joined below r_c = 5.25 (1.05 times the
    rods' contact distance 5, as 2.1 is for the paper's beads of diameter 2),
    electrodes at x 68 and 188.  This deposit percolates between the
    electrodes.  Timed per lb_kirchhoff call (neighbour scan, solve,
    currents, copy-out; the workspace is the caller's)."""
    import torch

    from paper_2607_06794_amd import inputs
    from paper_2607_06794_amd.sim import Lattice, kirchhoff
    from tests import cases

    rods = inputs.deposit_rods(n_rods, (40.0, 216.0), (4.0, 124.0), 3.5, seed=seed)
    lp = rod_params(cases.lattice_params(case, "f32"))
    lat = Lattice(lp, case["rho"], case["mat"], rods=rods)
    pos = lat.rod_beads(2.0)
    torch.cuda.synchronize()
    lat.close()
    spec = dict(r_c=5.25, x_src=68.0, x_snk=188.0)
    o = kirchhoff(pos, **spec)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        o = kirchhoff(pos, **spec)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) / reps * 1e3
    res = {"deposit": f"{n_rods} crossed rods on the substrate (seed {seed})", "beads": int(pos.shape[0]),
           "bead_spacing": 2.0, **spec, "edges": o["edges"], "max_degree": o["max_degree"],
           "iterations": o["iterations"], "rel_residual": o["rel_residual"], "I_tot": o["I_tot"],
           "kappa": o["kappa"], "ms_per_solve": ms}
    return res, pos.cpu().numpy()


def cg_form(steps=200, warmup=20):
    """The paper's colour-gradient step (four passes: stream with colour and
    moments, ghost colours of the walls, normals, then collision with the
    capillary force and recolouring) on the same cap under a lid (the step
    takes no reservoir), FP32: 150 / 60 / 120 degrees on stripe / surround /
    lid, sigma = 0.01, beta = 0.7.  Timed per step with HIP events on the
    launch stream; bytes per fluid node: the method's minimum 304 (each
    population read and written once) and the passes' 388 (besides, C written
    once and read twice, rho_k and j, the normal and |grad C| written once and
    read once)."""
    import torch

    from paper_2607_06794_amd import inputs
    from paper_2607_06794_amd.sim import Lattice, LatticeParams
    from tests import cases

    spec = inputs.CapSpec()
    c = cases.sink_case(shape=spec.shape, footprint=spec.footprint, height=spec.height, stripe=spec.stripe,
                        seed=spec.seed, J0=0.0, K=0.01)
    rho = c["rho"].copy()
    th = np.full(9, np.pi / 2)
    th[inputs.STRIPE], th[inputs.SURROUND] = np.deg2rad(60.0), np.deg2rad(120.0)
    lp = LatticeParams(shape=c["shape"], periodic=c["periodic"], prec="f32", model="cg", cg_sigma=0.01, cg_beta=0.7,
                       cg_grad_eps=1e-2, cg_theta=th)
    lat = Lattice(lp, rho, c["mat"])
    n_fluid = int(lat.observables()["fluid_nodes"])
    lat.step(warmup)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    lat.step(steps)
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    o = lat.observables(allow_unstable=True)
    lat.close()
    return {"us_per_step": ms * 1e3, "mlups": n_fluid / (ms * 1e-3) / 1e6, "fluid_nodes": n_fluid,
            "gbs_at_304": 304 * n_fluid / (ms * 1e-3) / 1e9, "gbs_at_388": 388 * n_fluid / (ms * 1e-3) / 1e9,
            "frac_at_388": 388 * n_fluid / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, "status": int(o["status"]),
            "note": "colour-gradient step, cap under a lid, FP32, four passes per step"}


def filament_form(steps=100, warmup=10):
    """The paper's bead-spring filaments (Eqs. 9-12) in the same cap: as many
    of 200 requested straight chains of twelve beads (L = 24) as fit inside
    the liquid, eps_coh = 0.004, FP32 fluid.  Timed with HIP events on the
    launch stream per coupled step (fluid step + filament update: gather,
    partner lists, five substeps, spread, apply) inside a call, and, on a fresh
    lattice, for calls of one fluid step and one filament update in turn."""
    import torch

    from paper_2607_06794_amd import inputs
    from paper_2607_06794_amd.sim import Lattice
    from tests import cases

    case = cases.cap_case()
    spec = inputs.CapSpec()
    beads = inputs.place_filaments(200, 12, 1.95, (256, 128, 64), inside=inputs.cap_inside(spec), seed=2600,
                                   clearance=2.2, margin=0.5, zmin=1.5, max_trials=300000)
    nf = len(beads) // 12
    lp = cases.lattice_params(case, "f32")
    lp.wall_z, lp.n_fil, lp.fil_beads, lp.fil_eps_coh = 0.5, nf, 12, 0.004
    lat = Lattice(lp, case["rho"], case["mat"], beads=beads)
    n_fluid = int(lat.observables()["fluid_nodes"])
    lat.coupled_step(warmup)
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    lat.coupled_step(steps)
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    o = lat.observables(allow_unstable=True)
    lat.close()
    lat = Lattice(lp, case["rho"], case["mat"], beads=beads)
    lat.coupled_step(warmup)
    torch.cuda.synchronize()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2 * steps + 1)]
    ev[0].record(stream)
    for s in range(steps):
        lat.step(1)
        ev[2 * s + 1].record(stream)
        lat.filament_step()
        ev[2 * s + 2].record(stream)
    torch.cuda.synchronize()
    mf = sum(ev[2 * s].elapsed_time(ev[2 * s + 1]) for s in range(steps)) / steps
    mu = sum(ev[2 * s + 1].elapsed_time(ev[2 * s + 2]) for s in range(steps)) / steps
    lat.close()
    return {"filaments": nf, "beads": nf * 12, "us_per_coupled_step": ms * 1e3, "us_single_fluid_step": mf * 1e3,
            "us_single_filament_update": mu * 1e3, "mlups": n_fluid / (ms * 1e-3) / 1e6, "status": int(o["status"]),
            "placement": "straight chains fully inside the cap (clearance 2.2, margin 0.5), of 200 requested"}


def cpu_baseline(case, sample_steps):
    from oracle import lbm
    from tests import cases

    run = lbm.Run(case["rho"], case["mat"], cases.oracle_params(case))
    n_fluid = int((case["mat"] == 0).sum())
    t0 = time.perf_counter()
    run.step(sample_steps)
    dt = time.perf_counter() - t0
    return n_fluid * sample_steps / dt / 1e6, dt


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=300)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--segment", type=int, default=100, help="coupled steps per freshly initialised segment")
    ap.add_argument("--prec", default="f32", choices=list(BYTES_PER_ELEM))
    ap.add_argument("--rounding", default="nearest", choices=["nearest", "stochastic"],
                    help="16-bit storage rounding of the timed lattice")
    ap.add_argument("--rho-ref", type=float, default=0.0, help="16-bit storage reference density of the timed lattice")
    ap.add_argument("--tile-y", type=int, default=0)
    ap.add_argument("--rows-per-thread", type=int, default=0)
    ap.add_argument("--zchunk", type=int, default=0)
    ap.add_argument("--cpu-steps", type=int, default=8, help="oracle steps in the CPU baseline sample (0: skip)")
    ap.add_argument("--rods", type=int, default=200, help="rods requested (stress placement)")
    ap.add_argument("--forms", type=int, default=1, help="also time the FP16/BF16 storage forms")
    ap.add_argument("--batched", type=int, default=64, help="lattices of the many-droplet sweep (0: skip)")
    ap.add_argument("--batched-steps", type=int, default=10)
    ap.add_argument("--surrogate", type=int, default=64, help="droplets for the surrogate data (0: skip)")
    ap.add_argument("--network", type=int, default=1, help="resistor network of the rods' beads (0: skip)")
    ap.add_argument("--surrogate-epochs", type=int, default=40)
    ap.add_argument("--surrogate-ensemble", type=int, default=12,
                    help="independent runs of the accuracy droplet for the ensemble deposit comparison (0: skip)")
    ap.add_argument("--surrogate-drift", type=float, default=0.5,
                    help="a jump moves each rod by this times its displacement over the interval before "
                         "(negative: rods held in place)")
    ap.add_argument("--surrogate-lambda", type=float, default=100.0,
                    help="weight of the squared relative rho_A mass error in the training loss")
    ap.add_argument("--surrogate-snapshots", type=int, default=16,
                    help="canvases per droplet (pairs: 7/8 of the droplets x (snapshots - 1))")
    ap.add_argument("--tile-cache", default=None, help="not used: tau = 1 has no tiles")
    ap.add_argument("--unet-only", action="store_true", help="time the U-Net alone (one JSON line)")
    ap.add_argument("--copy-probe", type=int, default=0, help="MiB of a plain copy for counter calibration, then exit")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (asked for --gpus {args.gpus}); the library has no multi-GPU path",
              file=sys.stderr)
        sys.exit(2)

    import torch

    from tests import cases

    torch.cuda.init()
    if args.copy_probe:
        print(json.dumps(copy_probe(args.copy_probe)), flush=True)
        return
    if args.unet_only:
        print(json.dumps(unet_form()), flush=True)
        return
    from paper_2607_06794_amd import inputs

    case = cases.cap_case()
    spec = inputs.CapSpec()
    box = (256, 128, 64)
    # physical placement (fully immersed, non-overlapping) fits far fewer than
    # the requested count; the timed run places the requested count anywhere
    # in the fluid volume (stress placement) and reports both counts
    n_phys = len(inputs.place_rods(args.rods, 24.0, 2.0, box, inside=inputs.cap_inside(spec), seed=2000,
                                   max_trials=20000)) if args.rods else 0
    rods = inputs.place_rods(args.rods, 24.0, 2.0, box, inside=None, seed=2000, max_trials=20000) if args.rods else None
    n_rods = 0 if rods is None else len(rods)
    tile = dict(tile_y=args.tile_y, rows_per_thread=args.rows_per_thread, zchunk=args.zchunk)
    log(f"[bench] workload cap 256x128x64 prec={args.prec} rods={n_rods} (physical fit {n_phys}) "
        f"steps={args.steps} warmup={args.warmup}")
    ms, ms_single, n_fluid, obs, nseg = time_step(case, args.prec, args.steps, args.warmup, tile, rods,
                                                  args.segment, rho_ref=(args.rho_ref, args.rho_ref),
                                                  rounding=args.rounding)
    mlups = n_fluid / (ms * 1e-3) / 1e6
    # the fluid's share: the same lattice without rods in calls of the same length;
    # the roofline's fluid step: in a call of 100 steps
    call = min(args.steps, args.segment) if args.segment > 0 else args.steps
    (ms_fluid, _, n_free, _, _), (ms_inner, _, _, _, _) = (
        time_step(case, args.prec, n, args.warmup, tile, rho_ref=(args.rho_ref, args.rho_ref), rounding=args.rounding)
        for n in (call, 100))
    bpl = step_bytes_per_lu(args.prec, args.rho_ref)
    achieved = bpl * n_free / (ms_inner * 1e-3) / 1e9
    log(f"[bench] {ms * 1e3:.1f} us/step (fluid without rods {ms_fluid * 1e3:.1f}, fluid step in a call of its own "
        f"{ms_single * 1e3:.1f}), {mlups:.0f} MLUPS, {achieved:.0f} GB/s in the fluid step")

    forms = {}
    if args.forms:
        # storage forms on the same lattice, fluid only, against plain FP32;
        # each 16-bit form also states its error against the oracle (10^4
        # steps of the static droplet)
        errs = storage_error_report()
        base, base1, n_form, _, _ = time_step(case, "f32", 500, 50, tile)

        def rates(msf, msk, n, prec):
            # a step inside a call of many, and a step in a call of its own
            # (from populations to populations: the algorithmic bytes)
            return {"us_per_step": msf * 1e3, "us_per_single_step": msk * 1e3, "mlups": n / (msf * 1e-3) / 1e6,
                    "speedup_vs_f32": base / msf, "speedup_vs_f32_single": base1 / msk,
                    "gbs_algorithmic_single": algorithmic_bytes_per_lu(prec) * n / (msk * 1e-3) / 1e9}

        forms["f32"] = rates(base, base1, n_form, "f32")
        for name, (prec, ref) in FORMS16.items():
            msf, msk, _, _, _ = time_step(case, prec, 500, 50, tile, rho_ref=(ref, ref), rounding="stochastic")
            forms[name] = {"storage": "FP16" if prec == "f16dev" else "BF16", "rho_ref": ref, "rounding": "stochastic",
                           "stores": "f_i" if ref == 0 else "f_i - w_i rho_ref (deviation from the lattice weights)",
                           **rates(msf, msk, n_form, prec), "error_vs_oracle": errs[name]}
            log(f"[bench] form {name}: {msf * 1e3:.1f} us, {forms[name]['mlups']:.0f} MLUPS, "
                f"x{forms[name]['speedup_vs_f32']:.2f} vs f32 (x{forms[name]['speedup_vs_f32_single']:.2f} with one step "
                f"per call)")
        # the paper's evaporation law (Eq. 8) in place of the reservoir plane:
        # the same cap under a lid, FP32, J0 = 1e-4, K = 0.01, h0 = the cap height
        sink_case = cases.sink_case(shape=case["shape"], footprint=spec.footprint, height=spec.height,
                                    stripe=spec.stripe, seed=spec.seed, J0=1e-4, K=0.01)
        msf, msk, n_sink, obs_s, _ = time_step(sink_case, "f32", 500, 50, tile)
        forms["f32sink"] = {**rates(msf, msk, n_sink, "f32"),
                            "moved_A_to_B": float(obs_s["ledger"][0]), "status": int(obs_s["status"]),
                            "note": "interfacial sink (Eq. 8) instead of the reservoir plane, lid on top, 550 steps"}
        log(f"[bench] form f32sink: {msf * 1e3:.1f} us, {forms['f32sink']['mlups']:.0f} MLUPS, "
            f"x{forms['f32sink']['speedup_vs_f32']:.2f} vs f32, moved {obs_s['ledger'][0]:.1f}")

    if args.forms:
        forms["f32cg"] = cg_form()
        log(f"[bench] form f32cg: {forms['f32cg']['us_per_step']:.1f} us, {forms['f32cg']['mlups']:.0f} MLUPS")
        forms["f32filaments"] = filament_form()
        ff = forms["f32filaments"]
        log(f"[bench] form f32filaments: {ff['filaments']} chains, {ff['us_per_coupled_step']:.1f} us per coupled "
            f"step (in calls of one: fluid {ff['us_single_fluid_step']:.1f} + filaments "
            f"{ff['us_single_filament_update']:.1f})")

    batched = None
    if args.batched > 0:
        log(f"[bench] batched form: {args.batched} droplets of the sweep")
        batched = batched_form(args.batched_steps, 2, args.batched)

    sur = None
    if args.surrogate > 0:
        log(f"[bench] surrogate form: {args.surrogate} droplets")
        sur = surrogate_form(args.surrogate, n_snap=args.surrogate_snapshots, epochs=args.surrogate_epochs,
                             lam=args.surrogate_lambda, n_ens=args.surrogate_ensemble, drift=args.surrogate_drift,
                             log_fn=log)

    net, net_pos = None, None
    if args.network > 0:
        net, net_pos = network_form(case)
        log(f"[bench] network: {net['beads']} beads, {net['edges']} edges, {net['iterations']} CG iterations, "
            f"kappa* {net['kappa']:.4g}, {net['ms_per_solve']:.2f} ms per solve")

    cpu = None
    if args.cpu_steps > 0:
        log(f"[bench] cpu baseline: oracle, {args.cpu_steps} steps of the same lattice")
        v, dt = cpu_baseline(case, args.cpu_steps)
        cpu = {"value": v, "unit": "MLUPS", "cores": 1, "kind": "oracle",
               "sample": f"{args.cpu_steps} FP64 NumPy oracle steps of the full 256x128x64 cap from t=0 "
                         f"({dt:.1f} s, 1 of {os.cpu_count()} host cores)"}
        if net_pos is not None:
            from oracle import network as onet

            t0 = time.perf_counter()
            o = onet.kirchhoff(net_pos, net["r_c"], net["x_src"], net["x_snk"])
            cpu["network"] = {"ms_per_solve": (time.perf_counter() - t0) * 1e3, "kind": "oracle",
                              "I_tot": o["I_tot"], "edges": o["edges"]}

    tr = traffic_record(args.prec, n_free, ms_inner) if args.rho_ref == 0.0 else None
    out = {
        "metric": METRIC,
        "value": mlups,
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": args.prec,
        "data": "synthetic",
        "config": {
            "workload": "elongated sessile cap 256x128x64, Shan-Chen D3Q19 two-component, G=3.6, tau=1, "
                        "striped bounce-back wall, reservoir plane (rho_A=0), rigid rods L=24 R=2 eps=1e-4; "
                        "one step = fluid step + rod update",
            "lattice": [256, 128, 64],
            "fluid_nodes": n_fluid,
            "prec": args.prec,
            "rods": n_rods,
            "rods_placement": "stress (requested count anywhere in the fluid)",
            "rods_physical_fit": n_phys,
            "timed_segments": nseg,
            "us_fluid_step": ms_fluid * 1e3,
            "us_single_fluid_step": ms_single * 1e3,
            "rod_time_share": max(0.0, 1.0 - ms_fluid / ms),
        },
        "forms": forms,
        "batched": batched,
        "surrogate": sur,
        "network": net,
        "roofline": {
            "bound": "hbm",
            "achieved": achieved,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS,
            "traffic": (tr["gbs"] if tr else None),
            "traffic_bytes_per_step": (tr["bytes_per_step"] if tr else None),
            "traffic_vs_needed": (tr["vs_needed"] if tr else None),
            "kernel": ("sc_stream_state_kernel + sc_collide_kernel" if args.prec in ("f32", "f64")
                       else "sc_stream_kernel + sc_collide_kernel"),
            "bytes_per_lu": bpl,
            "units_per_step": n_free,
            "algorithmic_bytes_per_lu_single": algorithmic_bytes_per_lu(args.prec),
            "achieved_single": algorithmic_bytes_per_lu(args.prec) * n_fluid / (ms_single * 1e-3) / 1e9,
        },
        "cpu_baseline": cpu,
        "status": int(obs["status"]),
    }
    print(json.dumps(_finite(out), allow_nan=False), flush=True)


if __name__ == "__main__":
    main()
