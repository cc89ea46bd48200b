"""Pins of the oracle's cell words at the ends of their ranges."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import sim
from oracle.model import PROLIF
from oracle.philox import INIT_STEP, site_words


@pytest.mark.parametrize("A0", [16, 256, 257, 1000, 9000, 70000])
def test_initial_ages_saturate(params, A0):
    """Seeded words hold PROLIF and min(floor(w0 A0 / 2^32), 255), nothing else."""
    _, cells = sim.init_state(replace(params, A0=A0), 64, 1, 2, 5)
    ys, xs = np.nonzero(cells)
    w0 = site_words(ys * 64 + xs, INIT_STEP, 2, 1, 5)[0].astype(object)
    age = np.array([min(int(w) * A0 >> 32, 255) for w in w0])
    assert len(ys) == 113 and np.array_equal(cells[ys, xs], PROLIF | (age << 2))
