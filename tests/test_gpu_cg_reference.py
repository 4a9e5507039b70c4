"""The colour-gradient step's densities with a storage reference: a component that
is nearly absent (0.5 to 2 percent) keeps the precision of its stored
populations.

One FP32 step against FP64 without interface normals.  A stored deviation is
rounded to half a last place of w_i rho_ref (rms 0.29 of a last place: 8.6e-9 for
the rest population, 1.1e-9 and 0.5e-9 for the others), once at the start and once
after the step: 1.4e-8 rms in a density; the rest of the step works on numbers of a
hundredth.  Bound: 2.5e-8 (the sum of the deviations has 6e-8)."""
import numpy as np
import pytest

from tests import cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau", [(1.0, 1.0), (0.9, 1.0)])
@pytest.mark.parametrize("ref", [0.0, 1.0])
def test_nearly_absent_component(tau, ref):
    from paper_2607_06794_amd.sim import Lattice

    shape = (12, 18, 40)
    z, y, x = np.meshgrid(*(np.arange(n) for n in shape), indexing="ij")
    few = (20 + (7 * x + 13 * y + 29 * z) % 61) / 4096.0
    rho = np.stack([few, 1.0 - few])
    out = {}
    for prec in ("f64", "f32"):
        print(f"[gpu] colour gradient, rho_ref={ref} tau={tau} {prec}", flush=True)
        c = dict(shape=shape, periodic=(True, True, True), G=0.0, tau=tau, body_force=(0.0, 0.0, 0.0),
                 evaporation=False)
        lp = cases.lattice_params(c, prec, rho_ref=(ref, ref))
        lp.model, lp.cg_sigma, lp.cg_grad_eps, lp.cg_theta = "cg", 0.01, 10.0, np.full(9, np.pi / 2)
        lat = Lattice(lp, rho, np.zeros(shape, np.uint8))
        lat.step(1)
        out[prec] = lat.export()[0][0]
        lat.close()
    rms = float(np.sqrt(np.mean((out["f32"] - out["f64"]) ** 2)))
    print("rms", rms, flush=True)
    assert abs(out["f64"].sum() - few.sum()) < 1e-9 and rms <= 2.5e-8
