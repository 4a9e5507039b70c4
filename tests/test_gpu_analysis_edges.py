"""The split column scan, the block-wise reductions and the contact graph at the
sizes where their splits can go wrong, against the FP64 oracle: planes fewer
than, equal to and one more than the scan's runs, columns off the multiples of
64, wet runs that end at the lattice's edges, and chains of rods longer than
one step of the labels' propagation.  Lengths and angles to 1e-9, counts and
labels exactly."""
import numpy as np
import pytest

from oracle import lbm
from oracle import observables as OB
from paper_2607_06794_amd import inputs
from tests import cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(3, 5, 7), (15, 9, 64), (16, 8, 65), (17, 7, 63), (33, 3, 130)])
def test_droplet_shape(shape):
    from paper_2607_06794_amd.sim import Lattice

    nz, ny, nx = shape
    rng = np.random.default_rng(nz)
    mat = np.zeros(shape, np.uint8)
    mat[0] = inputs.STRIPE
    mat[-1] = inputs.SURROUND
    z, y, x = np.meshgrid(*(np.arange(n) for n in shape), indexing="ij")
    c = np.clip(0.9 * (1.3 - z / (0.6 * nz) - np.abs(x - nx // 2) / nx), -0.9, 0.9) + 0.05 * rng.random(shape)
    rho = np.stack([0.5 * (1 + c), 0.5 * (1 - c)])
    rho[:, mat != 0] = 0.0
    case = dict(shape=shape, periodic=(True, True, False), G=0.0, tau=(1.0, 1.0), rho=rho, mat=mat, evaporation=False,
                body_force=(0.0, 0.0, 0.0))
    print(f"[gpu] droplet shape {shape}", flush=True)
    lat = Lattice(cases.lattice_params(case, "f64"), rho, mat)
    xc, yc = float(nx // 2), float(ny // 2)
    g = lat.droplet_shape(xc, yc)
    obs = lat.observables()
    lat.close()
    run = lbm.Run(rho, mat, cases.oracle_params(case))
    o = OB.droplet_shape(lbm.fields(run.f, run.material)[0], mat, xc, yc)
    assert g["wet_nodes"] == o.wet_nodes and obs["fluid_nodes"] == int((mat == 0).sum())
    for k in ("height", "r_x", "r_y", "theta_x", "theta_y"):
        assert abs(g[k] - getattr(o, k)) <= 1e-9, (k, g[k], o)
    assert np.abs(obs["mass"] - run.masses()).max() <= 1e-12 * run.masses().max()


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130])
def test_contact_graph_of_a_chain(n):
    """Rods along x touching end to end in shuffled order: one cluster whose
    label travels the whole chain; and the same chain cut in the middle."""
    from paper_2607_06794_amd.sim import Lattice

    half, gap = 2.0, 4.5  # L = 8, R = 2; neighbours' segments 0.5 apart
    nx = int(gap * n) + 24
    rng = np.random.default_rng(n)
    perm = rng.permutation(n)
    for cut in (False, True):
        rods = np.zeros((n, 13))
        xs = 10.0 + gap * np.arange(n) + (3.0 if cut else 0.0) * (np.arange(n) >= (n + 1) // 2)
        rods[perm, 0] = xs
        rods[:, 1], rods[:, 2] = 6.0, 6.0
        rods[:, 3:7] = (np.sqrt(0.5), 0.0, np.sqrt(0.5), 0.0)  # e_z to e_x
        mat = np.zeros((12, 12, nx), np.uint8)
        mat[0] = mat[-1] = inputs.SURROUND
        rho = np.ones((2,) + mat.shape) * 0.5
        rho[:, mat != 0] = 0.0
        case = dict(shape=mat.shape, periodic=(True, True, False), G=0.0, tau=(1.0, 1.0), rho=rho, mat=mat,
                    evaporation=False, body_force=(0.0, 0.0, 0.0))
        lp = cases.lattice_params(case, "f64")
        lp.rod_length, lp.rod_radius = 2 * half + 4.0, 2.0
        print(f"[gpu] contact graph of {n} rods, cut={cut}", flush=True)
        lat = Lattice(lp, rho, mat, rods=rods)
        d = lat.deposit(8, 4, nx / 2.0, 6.0, float(nx), 12.0, r_contact=1.0, x_src=10.0, x_snk=xs[-1])
        lat.close()
        left = perm[: (n + 1) // 2] if cut else perm
        right = perm[(n + 1) // 2:] if cut else perm[:0]
        labels = np.empty(n, int)
        for part in (left, right):
            if len(part):
                labels[part] = part.min()
        assert np.array_equal(d["labels"], labels)
        assert d["edges"] == (n - 1 if not cut else n - 1 - (len(right) > 0))
        assert d["largest"] == max(len(left), len(right))
        assert d["spanning"] == (not cut or len(right) == 0)
