"""The coefficient's per-sample extremes at every number of x factors the
kernel is compiled for, at sample counts past one grid dimension, and on
values that are not finite."""
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


# short correlation lengths rank low products of many 1D modes first, long
# ones single high modes: 1, 2, 3, 4 and up to 6 different x factors.  The sum
# of M + 1 terms in another order differs by at most 2 (M + 3) 2^-53 of the
# terms' magnitudes, which sigma sum sqrt(lambda) |phi|^3 < 16 bounds; the
# tables mirror about the middle of the axis to the same rounding.
@pytest.mark.parametrize("N,s,M,L", [(1, 1, 1, 1.0), (2, 3, 2, 1.0), (7, 5, 4, 1.0), (12, 40, 10, 1.0),
                                     (9, 6, 16, 0.05), (9, 6, 16, 1.0), (9, 6, 16, 50.0), (33, 3, 10, 1.0)])
def test_extrema_match_oracle(E, N, s, M, L):
    from oracle import oracle as orc
    xi = draw_xi(100 * N + s, s, M)
    kl = E.kl_build(N, M, L)
    kmin, kmax = E.kl_extrema(N, kl, torch.as_tensor(xi, device=DEV), M, 0.4, L=L)
    omin, omax = orc.sample_extrema(N, M, L, 1.0, 0.4, xi)
    tol = 2 * 20 * 2.0 ** -53 * 16 * 4
    assert np.abs(kmin.cpu().numpy() - omin).max() <= tol and np.abs(kmax.cpu().numpy() - omax).max() <= tol


def test_extrema_of_many_samples(E):
    from oracle import oracle as orc
    N, s, M = 2, 65535 + 300, 3
    xi = draw_xi(9, s, M)
    kl = E.kl_build(N, M)
    kmin, kmax = E.kl_extrema(N, kl, torch.as_tensor(xi, device=DEV), M, 0.4)
    at = np.array([0, 1, 65534, 65535, 65536, s - 1])
    omin, omax = orc.sample_extrema(N, M, 1.0, 1.0, 0.4, xi[at])
    assert np.abs(kmin.cpu().numpy()[at] - omin).max() <= 1e-13
    assert np.abs(kmax.cpu().numpy()[at] - omax).max() <= 1e-13


def test_extrema_of_values_that_are_not_finite(E):
    N, M = 6, 4
    xi = draw_xi(11, 5, M)
    xi[1, 0] = np.inf       # the first mode is positive everywhere: +inf at every point
    xi[2, 0] = -np.inf
    xi[3, 1] = np.inf       # the second changes sign: -inf to +inf
    xi[4, :2] = np.inf, np.nan
    kl = E.kl_build(N, M)
    kmin, kmax = (t.cpu().numpy() for t in E.kl_extrema(N, kl, torch.as_tensor(xi, device=DEV), M, 0.4))
    assert np.isfinite(kmin[0]) and np.isfinite(kmax[0])
    assert kmin[1] == np.inf and kmax[1] == np.inf and kmin[2] == -np.inf and kmax[2] == -np.inf
    assert kmin[3] == -np.inf and kmax[3] == np.inf
    assert np.isnan(kmin[4]) and np.isnan(kmax[4])
    # coefficients near the largest number: the sums may pass it, not fault
    big = E.kl_extrema(N, kl, torch.full((2, M), 1e308, dtype=torch.float64, device=DEV), M, 3.0)
    assert not any(bool(torch.isfinite(t).all()) for t in big)
