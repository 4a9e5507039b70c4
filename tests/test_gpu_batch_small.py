"""Batches of lattices that keep populations alone but moments together (more than
64 MiB of populations in all): calls of several steps against each lattice stepped
by itself, one step per call, bit for bit."""
import numpy as np
import pytest

from paper_2607_06794_amd import inputs
from tests import cases

pytestmark = pytest.mark.gpu

SHAPES = {"f32": [(64, 64, 64), (31, 63, 65), (48, 48, 49)], "f64": [(48, 48, 48), (31, 49, 63), (33, 40, 47)]}


def spec(shape, walls):
    rho, mat = inputs.sphere_droplet(shape, min(shape) / 4, seed=3)
    if walls:
        mat[0], mat[-1] = inputs.STRIPE, inputs.SURROUND
        rho[:, mat != 0] = 0.0
    return dict(shape=shape, periodic=(True, True, not walls), G=1.8, tau=(1.0, 1.0), rho=rho, mat=mat,
                evaporation=False, body_force=(1e-5, 0.0, -1e-5))


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("graph", [True, False])
def test_small_lattices_together(prec, graph):
    from paper_2607_06794_amd.sim import Batch, Lattice

    specs = [spec(s, walls=k == 1) for k, s in enumerate(SHAPES[prec])]
    size = [38 * int(np.prod(s)) * (4 if prec == "f32" else 8) for s in SHAPES[prec]]
    assert max(size) < 64 << 20 < sum(size)
    lattices = lambda: [Lattice(cases.lattice_params(c, prec), c["rho"], c["mat"]) for c in specs]
    calls = [5, 2, 1, 4, 3]
    print(f"[gpu] batch of small lattices {prec} graph={graph}", flush=True)
    solo, lats = lattices(), lattices()
    for lat in solo:
        for _ in range(sum(calls)):
            lat.step(1)
    batch = Batch(lats)
    for n in calls:
        batch.step(n, rods=False, graph=graph)
        lats[1].observables(allow_unstable=True)
    for a, b in zip(solo, lats):
        fa, fb = a.export()[1], b.export()[1]
        assert np.abs(fa).max() > 0.01 and np.array_equal(fa, fb)
        oa, ob = a.observables(), b.observables()
        assert oa["status"] == ob["status"] and oa["step"] == ob["step"]
    batch.close()
    for lat in solo + lats:
        lat.close()
