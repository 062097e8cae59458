"""Rounding of the assemblies' diagonals, which are minus the sum of their row's
other entries: rows whose neighbours are all interior, against the 80-bit sum of
the 26 entries stored.

A rounding is at most u = 2^-53 of its result, u / sqrt 3 in the mean square.
Nine lines of three, three planes of three lines and the planes have results of
at most 1/9 (18 sums), 1/3 and 2/9 (three sums each) and 1 and 2/3 of the
entries' magnitudes S: sqrt(18 / 81 + 3 / 9 + 3 * 4 / 81 + 1 + 4 / 9) / sqrt 3 = 0.85
u S in the mean square at most."""
import numpy as np
import pytest
import torch

from workloads import draw_xi

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def E():
    from paper_1511_03703_amd import ens
    ens.lib()
    return ens


@pytest.mark.parametrize("kind", ["linear", "nonlinear"])
@pytest.mark.parametrize("N,s", [(11, 4), (14, 16), (16, 32)])
def test_diagonals(E, kind, N, s):
    M, sigma = 10, 0.2
    g, kl = E.graph_build(N), E.kl_build(N, M)
    xi = torch.as_tensor(draw_xi(9, s, M), device=DEV)
    if kind == "linear":
        v = E.assemble(g, kl, xi, M, sigma)[0]
    else:
        prob = E.nl_problem(M, sigma, 5.0, 0.0, (0.6, -0.3, 0.74))
        v = E.nl_assemble(g, kl, xi, prob, torch.ones((g.n, s), dtype=torch.float64, device=DEV))[1]
    v, rp = v.cpu().numpy(), g.row_ptr.cpu().numpy()
    i = np.arange(2, N - 1)
    rows = (i[:, None, None] * (N + 1) + i[None, :, None]) * (N + 1) + i[None, None, :]
    r = v[rp[rows.ravel()][:, None] + np.arange(27)].astype(np.longdouble)
    diag, off = r[:, 13], np.delete(r, 13, axis=1)
    err = (diag + off.sum(1)) / np.abs(off).sum(1)
    assert float(np.sqrt((err ** 2).mean())) <= 0.85 * 2.0 ** -53
