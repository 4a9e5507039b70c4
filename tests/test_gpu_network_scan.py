"""Networks beyond the row-sorted solve's size, whose neighbour scan takes four
beads per wavefront: every remainder of four, against the oracle."""
import numpy as np
import pytest

from tests.test_gpu_network import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8194, 8195, 8196, 8257])
def test_remainders(n):
    rng = np.random.default_rng(n)
    box = np.array([40.0, 12.0, 6.0]) * (n / 600.0) ** (1.0 / 3.0)
    pos = rng.uniform(0.0, 1.0, (n, 3)) * box
    pos[n - n // 9:, 1] += 1000.0 + 10.0 * np.arange(n // 9)  # the last beads have no neighbour
    pos[-2:] = pos[:2] + [0.5, 0.0, 0.0]  # but the very last do
    compare(pos, 2.1, 0.2 * box[0], 0.8 * box[0])
