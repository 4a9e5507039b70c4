"""Steps that the autotuner takes.

With tau = 1 the step is two untiled passes: the present shape alone is timed,
1 + trial_steps real steps, and stays.  With tau != 1 every supported shape is
(4 and 8 rows of one row per thread, by the z chunks that fit).
"""

import pytest

from tests import cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau1,shape", [(True, (8, 1)), (True, (16, 2)), (False, (8, 1))])
def test_steps_taken_and_shape_kept(tau1, shape, tmp_path):
    from paper_2607_06794_amd.sim import Lattice

    c = cases.cap_case(shape=(16, 20, 48), footprint=(30.0, 10.0), height=7.0, stripe=(34, 14))
    if not tau1:
        c = dict(c, tau=(0.9, 0.8))
    ty, rp = shape
    lat = Lattice(cases.lattice_params(c, "f32", tile_y=ty, rows_per_thread=rp, zchunk=5), c["rho"], c["mat"])
    t = lat.autotune(trial_steps=3, cache=str(tmp_path / "tiles.json"))
    steps = lat.observables()["step"]
    lat.close()
    assert t["us_per_step"] > 0 and not t["cached"]
    if tau1:
        assert steps == 4 and (t["tile_y"], t["rows_per_thread"], t["zchunk"]) == (ty, rp, 5)
    else:
        assert steps == 4 * 2 * 4  # chunks of 4, 8, 12 and 16 planes
