"""Steps of one call pass the state on as moments: the results are those of the
same steps taken one call at a time, bit for bit (populations, ledgers, rods).

Shapes at the edges of the bricks of 32 x 4 x 2 nodes: smaller than one, one
more and one less than a multiple, closed in x and y; calls of two steps (no
step between the first and the last), odd and even; a storage reference density;
with rods, ones that leave the wall so that nodes next to it are uncovered
(these return their own populations from the wall, whichever way they are kept)."""
import numpy as np
import pytest

from oracle import lbm
from oracle import rods as R
from paper_2607_06794_amd import inputs
from tests import cases

pytestmark = pytest.mark.gpu

SHAPES = [(4, 3, 3), (5, 5, 33), (4, 4, 32), (7, 9, 65), (6, 17, 31), (5, 40, 97)]


def make(shape, closed):
    nz, ny, nx = shape
    rng = np.random.default_rng(nx)
    mat = np.zeros(shape, np.uint8)
    mat[0] = inputs.SURROUND
    mat[0, :, : nx // 2] = inputs.STRIPE
    mat[-1] = inputs.GHOST
    if closed:
        mat[:-1, 0], mat[:-1, -1], mat[:-1, :, 0], mat[:-1, :, -1] = 4, 5, 6, 7
    x = np.arange(nx)[None, None, :]
    a = 0.5 + 0.4 * np.cos(2 * np.pi * x / nx) + 0.02 * rng.random(shape)
    rho = np.stack([a, 1.05 - a + 0.02 * rng.random(shape)])
    rho[:, mat != 0] = 0.0
    return dict(shape=shape, periodic=(not closed, not closed, False), G=1.2, tau=(1.0, 1.0), rho=rho, mat=mat,
                evaporation=True, body_force=(1e-5, 0.0, -2e-5))


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("prec,ref,closed", [("f64", 0.0, False), ("f64", 0.5, True), ("f32", 1.0, False),
                                             ("f32", 0.0, True)])
def test_one_call_is_many(shape, prec, ref, closed):
    from paper_2607_06794_amd.sim import Lattice

    if closed and min(shape[1:]) < 4:
        closed = False
    c = make(shape, closed)
    out = []
    print(f"[gpu] steps of one call {shape} {prec} rho_ref={ref} closed={closed}", flush=True)
    for calls in ([1] * 9, [9], [2, 3, 4]):
        lat = Lattice(cases.lattice_params(c, prec, rho_ref=(ref, ref)), c["rho"], c["mat"])
        for n in calls:
            lat.step(n)
        out.append((lat.export()[1], lat.observables(allow_unstable=True)))
        lat.close()
    run = lbm.Run(c["rho"], c["mat"], cases.oracle_params(c))
    run.step(9)
    assert cases.rel_err(out[0][0], run.f) <= (1e-12 if prec == "f64" else 1e-5)
    for f, o in out[1:]:
        assert np.array_equal(f, out[0][0])
        assert np.array_equal(o["ledger"], out[0][1]["ledger"]) and o["status"] == out[0][1]["status"]


@pytest.mark.parametrize("prec,n", [("f64", 62), ("f32", 78)])
def test_without_reservoir(prec, n):
    """Periodic, just above the size from which such a lattice takes moments."""
    from paper_2607_06794_amd.sim import Lattice

    rho, mat = inputs.sphere_droplet((n, n, n), n / 4, seed=3)
    c = dict(shape=(n, n, n), periodic=(True,) * 3, G=3.6, tau=(1.0, 1.0), rho=rho, mat=mat, evaporation=False,
             body_force=(0.0, 0.0, 0.0))
    out = []
    for calls in ([1] * 5, [5], [2, 3]):
        print(f"[gpu] steps of one call {n}^3 {prec} {calls}", flush=True)
        lat = Lattice(cases.lattice_params(c, prec), rho, mat)
        for k in calls:
            lat.step(k)
        out.append(lat.export()[1])
        lat.close()
    assert np.array_equal(out[1], out[0]) and np.array_equal(out[2], out[0])


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_coupled_call_is_many(prec):
    """A rod leaves the wall it touches, another crosses the liquid."""
    from paper_2607_06794_amd.sim import Lattice
    from tests import test_gpu_rods as TR

    shape = (20, 24, 40)
    spec = inputs.CapSpec(shape=shape, footprint=(24.0, 12.0), height=8.0, stripe=(28, 14))
    rho, mat = inputs.sessile_cap(spec)
    c = dict(shape=shape, periodic=(True, True, False), G=3.6, tau=(1.0, 1.0), rho=rho, mat=mat, evaporation=True,
             body_force=(0.0, 0.0, 0.0))
    q = np.sqrt(0.5)
    rods = np.zeros((2, 13))
    rods[:, 3], rods[:, 5] = q, q  # along x
    rods[0, :3], rods[0, 7:10] = (20.0, 12.3, 2.9), (0.0, 0.15, 0.2)
    rods[1, :3], rods[1, 7:10] = (18.0, 5.2, 9.4), (0.02, 0.3, -0.05)
    lp = cases.lattice_params(c, prec)
    r = TR.ROD
    lp.rod_length, lp.rod_radius, lp.rod_rho = 12.0, 2.0, 4.0
    lp.eps_att, lp.eps_rep, lp.rod_d0, lp.rod_rcut = r["eps_att"], r["eps_rep"], r["d0"], r["r_cut"]
    lp.eps_wall, lp.rod_d0_wall, lp.n_sub, lp.wall_z = r["eps_wall"], r["d0_wall"], r["n_sub"], 0.5
    out = []
    for calls in (None, [9], [2, 3, 4]):
        print(f"[gpu] coupled steps of one call {prec} {calls}", flush=True)
        lat = Lattice(lp, rho, mat, rods=rods)
        if calls is None:
            for _ in range(9):
                lat.step(1)
                lat.rods_step()
        else:
            for n in calls:
                lat.coupled_step(n)
        out.append((lat.export()[1], lat.rods(), lat.observables(allow_unstable=True)))
        lat.close()
    # the oracle's rod starts among the nodes next to the wall and leaves them
    rp = R.RodParams(wall_z=0.5, **dict(TR.ROD, rho_rod=4.0))
    nz, ny, nx = shape
    orods = R.Rods(rods[:, :3], rods[:, 3:7], rods[:, 7:10], rods[:, 10:13], rp, (nx, ny, nz), c["periodic"])
    run = R.CoupledRun(rho, mat, cases.oracle_params(c), orods)
    assert np.any(run.material[1] == lbm.ROD)
    run.step(9)
    assert not np.any(run.material[1] == lbm.ROD)
    for f, s, o in out[1:]:
        assert np.array_equal(f, out[0][0]) and np.array_equal(s, out[0][1])
        assert np.array_equal(o["ledger"], out[0][2]["ledger"]) and np.array_equal(o["solid"], out[0][2]["solid"])


@pytest.mark.parametrize("graph", [True, False])
def test_batch_call_is_many(graph):
    """Lattices of a batch that all keep moments: calls of 2 to 7 steps (from
    either buffer, replayed graphs with work between them) against each alone."""
    from paper_2607_06794_amd.sim import Batch
    from tests import test_gpu_batch as TB
    from tests import test_gpu_rods as TR

    def lattices():
        a, b = TR.cap_rods_case(), TR.periodic_case()
        a.update(tau=(1.0, 1.0), tile={}, eps_att=2e-4)
        b.update(tau=(1.0, 1.0), tile={}, eps_att=1e-4)
        c = make((6, 17, 31), False)
        c.update(rods=None, wall=None, tile={})
        return [TB._make(s) for s in (a, b, c)]

    calls = [7, 2, 3, 1, 6, 5]
    print(f"[gpu] batch of moment lattices, graph={graph}", flush=True)
    solo = lattices()
    for lat in solo:
        for _ in range(sum(calls)):
            lat.step(1)
            lat.rods_step()
    want = [TB._state(lat) for lat in solo]
    lats = lattices()
    batch = Batch(lats)
    for n in calls:
        batch.step(n, rods=True, graph=graph)
        lats[0].observables(allow_unstable=True)
    got = [TB._state(lat) for lat in lats]
    batch.close()
    for lat in solo + lats:
        lat.close()
    for (fw, rw, ow), (fg, rg, og) in zip(want, got):
        assert np.array_equal(fw, fg) and np.array_equal(rw, rg)
        assert np.array_equal(ow["ledger"], og["ledger"]) and np.array_equal(ow["solid"], og["solid"])


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_filament_call_is_many(prec):
    """Chains in a walled cap under the reservoir: the nodes that take their
    impulses keep stored populations between the steps of a call."""
    from paper_2607_06794_amd.sim import Lattice, LatticeParams
    from tests import test_gpu_filaments as TF

    c = TF.CASES["cap"]()
    out = []
    for calls in (None, [12], [2, 3, 7]):
        print(f"[gpu] filament steps of one call {prec} {calls}", flush=True)
        lp = LatticeParams(shape=c["shape"], periodic=c["periodic"], prec=prec, psi_solid=cases.PSI_SOLID.copy(),
                           evaporation=True, rho_top=(0.0, 1.0), wall_z=c["wall"], n_fil=len(c["beads"]) // c["n_per"],
                           fil_beads=c["n_per"], fil_eps_coh=c["eps_coh"])
        lat = Lattice(lp, c["rho"], c["mat"], beads=c["beads"])
        if calls is None:
            for _ in range(12):
                lat.step(1)
                lat.filament_step()
        else:
            for n in calls:
                lat.coupled_step(n)
        out.append((lat.export()[1], lat.beads(), lat.observables(allow_unstable=True)))
        lat.close()
    assert np.abs(out[0][1][:, 9:12]).max() > 0.0  # impulses were handed over
    for f, b, o in out[1:]:
        assert np.array_equal(f, out[0][0]) and np.array_equal(b, out[0][1])
        assert np.array_equal(o["ledger"], out[0][2]["ledger"]) and o["status"] == out[0][2]["status"]
