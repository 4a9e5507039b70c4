"""16-bit storage: the stored bits of a run.

A stored value is an FP32 sum rounded to 16 bits, so a sum that rounds
differently in its last bit can store another neighbour, and the steps after it
carry the difference on (1e-4 of the populations within 20 steps).  The
digests are those of the one-pass step that the two passes replaced, so that a
run continued or repeated with the two passes is the same run.  Initial densities
are exact binary fractions, made without a random generator or a library
function."""
import hashlib

import numpy as np
import pytest

from tests import cases

pytestmark = pytest.mark.gpu

SHAPE = (11, 13, 70)  # more than one 64-node row, ragged in every direction
DIGESTS = {
    ("f16dev", 0.0, "nearest"): "36dadfbe7b4f9984f0ef3a0c04e2f7e3",
    ("f16dev", 1.0, "stochastic"): "4ec368ace7e7bba30846f4726b7c0b56",
    ("bf16dev", 0.0, "nearest"): "77bf88efa71385d1e281d078f03baea9",
    ("bf16dev", 1.0, "stochastic"): "58480295318134f738603ce0f0594fe9",
}


def populations(prec, ref, rounding):
    from paper_2607_06794_amd import inputs
    from paper_2607_06794_amd.sim import Lattice, LatticeParams

    z, y, x = np.meshgrid(*(np.arange(n) for n in SHAPE), indexing="ij")
    # a block of liquid on the wall in gas, with steps of 1/64 in both
    liquid = (z < 6) & (np.abs(x - 33) < 22) & (np.abs(y - 6) < 4)
    grain = ((7 * x + 13 * y + 29 * z) % 16) / 1024.0
    rho = np.stack([np.where(liquid, 1.0, 0.03125) + grain, np.where(liquid, 0.03125, 1.0) - grain])
    mat = np.zeros(SHAPE, np.uint8)
    mat[0] = np.where((x[0] > 10) & (x[0] < 56), inputs.STRIPE, inputs.SURROUND)
    mat[-1] = 1
    lat = Lattice(LatticeParams(shape=SHAPE, periodic=(True, True, False), prec=prec, G=3.6,
                                body_force=(1e-5, -2e-5, 3e-5), psi_solid=cases.PSI_SOLID.copy(), evaporation=True,
                                rho_top=(0.0, 1.0), rho_ref=(ref, ref), rounding=rounding, sr_seed=7), rho, mat)
    lat.step(6)
    f = lat.export()[1]
    lat.close()
    return f


@pytest.mark.parametrize("form", sorted(DIGESTS), ids=lambda f: f"{f[0]}-{f[1]:g}-{f[2]}")
def test_stored_bits_of_a_run(form):
    print(f"[gpu] stored bits {form}", flush=True)
    f = populations(*form)
    assert np.isfinite(f).all() and f.max() > 0.1
    got = hashlib.sha256((f + 0.0).tobytes()).hexdigest()[:32]  # + 0.0: both zeros alike
    print(form, got, flush=True)
    assert got == DIGESTS[form]
