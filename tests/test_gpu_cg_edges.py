"""The colour-gradient step at the edges of its blocks of 256 nodes: planes
smaller than a block, blocks that end inside a row, node counts below, at and
above multiples of a block and of a block per XCD, closed directions in x and y
(ghost colours on the corners and edges of the closed box), and a storage
reference density, with tau = 1 (moments between the passes) and without.

Populations against the FP64 oracle: within 1e-12 (FP64) and 1e-5 (FP32)
relative to the largest, as in the parity runs of the full step."""
import numpy as np
import pytest

from oracle import cg as OC
from tests import cases

pytestmark = pytest.mark.gpu


def make(shape, closed):
    nz, ny, nx = shape
    rng = np.random.default_rng(nx + 7 * ny)
    mat = np.zeros(shape, np.uint8)
    mat[0], mat[-1] = 2, 4
    mat[0, :, : nx // 2] = 3
    if closed:
        mat[:, 0], mat[:, -1], mat[:, :, 0], mat[:, :, -1] = 5, 6, 7, 5
    if min(ny, nx) > 6:
        mat[: nz // 2, 3:5, 3:5] = 2  # a pillar
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    ins = ((x / nx - 0.45) / 0.3) ** 2 + ((y / ny - 0.5) / 0.35) ** 2 + ((z / nz - 0.4) / 0.4) ** 2 <= 1.0
    a = np.where(ins, 1.0, 0.0)
    rho = np.stack([a, 1.0 - a]) + 0.02 * rng.random((2,) + shape)
    rho[:, mat != 0] = 0.0
    return rho, mat


SHAPES = [((4, 3, 3), False), ((4, 4, 4), True), ((5, 7, 9), False), ((8, 16, 16), False), ((7, 5, 131), True),
          ((9, 31, 33), True)]
FORMS = [("f64", (1.0, 1.0), 0.0), ("f64", (0.8, 1.0), 0.5), ("f32", (1.0, 1.0), 1.0), ("f32", (1.0, 0.9), 0.0)]


# FP64 only: a normal within 6e-4 of the wall's, whose tangential part FP32 holds to 1e-4
ILL = (7, 5, 131)


@pytest.mark.parametrize("shape,closed", SHAPES)
@pytest.mark.parametrize("prec,tau,ref", FORMS)
def test_block_edges_against_the_oracle(shape, closed, prec, tau, ref):
    from paper_2607_06794_amd.sim import Lattice, LatticeParams

    if prec == "f32" and shape == ILL:
        pytest.skip("ill-conditioned in FP32")
    rho, mat = make(shape, closed)
    theta = np.linspace(0.9, 2.2, 9)
    per, g, steps = (not closed, not closed, False), (1e-5, 0.0, -2e-5), 4
    print(f"[gpu] colour gradient {shape} closed={closed} {prec} tau={tau} rho_ref={ref}", flush=True)
    lp = LatticeParams(shape=shape, periodic=per, prec=prec, tau=tau, body_force=g, model="cg", cg_sigma=0.01,
                       cg_beta=0.7, cg_grad_eps=1e-2, cg_theta=theta, rho_ref=(ref, ref))
    lat = Lattice(lp, rho, mat)
    lat.step(1)
    lat.step(steps - 1)
    _, f = lat.export()
    lat.close()
    run = OC.CGRun(rho, mat, OC.CGParams(shape=shape, periodic=per, tau=tau, sigma=0.01, beta=0.7, body_force=g,
                                         theta=theta))
    run.step(steps)
    fluid = (run.material == 0)[None, None]
    assert np.abs(run.f).max() < 1.0  # a stable reference
    assert cases.rel_err(np.where(fluid, f, 0), np.where(fluid, run.f, 0)) <= (1e-12 if prec == "f64" else 1e-5)
