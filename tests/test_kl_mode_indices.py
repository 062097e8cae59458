"""Which 1D modes the leading 3D modes use: x index i first appears as mode
3 i + 1 of the ranking (after (0, 0, j), (0, j, 0) and (j, 0, 0) of every j < i,
and (0, 0, i) and (0, i, 0)) or later, so 16 modes have x indices up to 5 at
most, whatever the correlation length.  The grouping predictor's kernel is built
for that many."""
import numpy as np
import pytest


@pytest.mark.parametrize("L", [1e-6, 1e-3, 0.02, 0.3, 1.0, 10.0, 1e3])
def test_x_indices_of_the_leading_modes(orc, L):
    for M in range(1, 17):
        t = np.asarray(orc.kl_modes(M, L)[0])
        nx = int(t[:, 0].max()) + 1
        assert 3 * (nx - 1) + 1 <= M
        assert nx <= 6
