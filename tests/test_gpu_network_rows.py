"""The row-sorted network solve at the sizes where its layout can go wrong:
one bead, the edges of a wavefront and of each rows-per-thread count, the last
size it takes and the first of the general solve, and beads of degree 0 and of
the full 64 stored neighbours.  Against the FP64 oracle's direct solve, with
the tolerances of the other network tests."""
import numpy as np
import pytest

from tests.test_gpu_network import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 2049, 4096, 4097, 8192, 8193])
def test_sizes(n):
    # a bar of mean degree about 7 between the electrodes, its tail beads far
    # away from everything (degree 0)
    rng = np.random.default_rng(n)
    box = np.array([40.0, 12.0, 6.0]) * (max(n, 8) / 600.0) ** (1.0 / 3.0)
    pos = rng.uniform(0.0, 1.0, (n, 3)) * box
    pos[n - n // 9:, 1] += 1000.0 + 10.0 * np.arange(n // 9)
    compare(pos, 2.1, 0.2 * box[0], 0.8 * box[0])


def test_full_rows():
    # 65 beads pairwise within r_c (64 neighbours each), once on the source
    # side and once between the electrodes, next to a spanning chain
    rng = np.random.default_rng(5)
    clump = rng.uniform(-0.5, 0.5, (65, 3))
    chain = np.stack([np.arange(0.0, 30.1, 1.6), np.full(19, 50.0), np.zeros(19)], axis=1)
    pos = np.concatenate([clump + [1.0, 0, 0], chain, clump + [15.0, 0, 0]])
    d = np.linalg.norm(pos[:, None] - pos[None], axis=2)
    deg = ((d > 0) & (d < 2.0)).sum(1)
    assert deg.max() == 64
    _, o = compare(pos, 2.0, 3.0, 25.0)
    assert o["I_tot"] > 1e-3
