"""The two-pass step (tau = 1) at the sizes where its blocks of 256 nodes can
go wrong, against the FP64 oracle: planes smaller than a block (several planes,
the reservoir's among them, in one block), blocks that end inside a row, node
counts below, at and above multiples of a block, and a storage reference
density (the deviations' own moments between the passes).

Populations within 1e-12 (FP64) and 1e-5 (FP32) relative, ledgers within 1e-11
and 1e-5 of the largest, as in the parity runs of the full step."""
import numpy as np
import pytest

from oracle import lbm
from paper_2607_06794_amd import inputs
from tests import cases

pytestmark = pytest.mark.gpu


def make(shape, seed):
    """Wall below (stripe and surround), a pillar of wall, reservoir on top."""
    nz, ny, nx = shape
    rng = np.random.default_rng(seed)
    mat = np.zeros(shape, np.uint8)
    mat[0] = inputs.SURROUND
    mat[0, :, : nx // 2] = inputs.STRIPE
    mat[-1] = inputs.GHOST
    if min(ny, nx) > 4:
        mat[: nz // 2, 1:3, 2:4] = inputs.SURROUND
    x = np.arange(nx)[None, None, :]
    a = 0.5 + 0.4 * np.cos(2 * np.pi * x / nx) + 0.02 * rng.random(shape)
    rho = np.stack([a, 1.05 - a + 0.02 * rng.random(shape)])
    rho[:, mat != 0] = 0.0
    return dict(shape=shape, periodic=(True, True, False), G=1.2, tau=(1.0, 1.0), rho=rho, mat=mat, evaporation=True,
                body_force=(1e-5, 0.0, -2e-5))


@pytest.mark.parametrize("shape", [(4, 3, 3), (5, 7, 9), (6, 16, 16), (4, 16, 16), (7, 5, 131), (9, 31, 33)])
@pytest.mark.parametrize("prec,ref", [("f64", 0.0), ("f64", 0.5), ("f32", 0.0), ("f32", 1.0)])
def test_block_edges_against_the_oracle(shape, prec, ref):
    from paper_2607_06794_amd.sim import Lattice

    c = make(shape, 77)
    steps = 12
    print(f"[gpu] two-pass step {shape} {prec} rho_ref={ref}", flush=True)
    lat = Lattice(cases.lattice_params(c, prec, rho_ref=(ref, ref)), c["rho"], c["mat"])
    lat.step(1)
    lat.step(steps - 1)
    obs = lat.observables(allow_unstable=True)
    _, f = lat.export()
    lat.close()
    run = lbm.Run(c["rho"], c["mat"], cases.oracle_params(c))
    run.step(steps)
    tol, tol_led = (1e-12, 1e-11) if prec == "f64" else (1e-5, 1e-5)
    assert cases.rel_err(f, run.f) <= tol
    assert np.abs(obs["ledger"] - run.ledger).max() <= tol_led * np.abs(run.ledger).max()
