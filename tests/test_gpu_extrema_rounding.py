"""Rounding of the coefficient's extremes where they are close to kappa0: the
modes' sum is formed on its own and added to kappa0 once.  Against 80-bit sums
over the KL table's values: half an ulp of the result, at most 2^-53 of it, and
40 roundings of the modes' magnitudes (their products and sums, and the table's
mirror images, whose abscissae differ by a rounding that a mode's frequency,
under 10 here, magnifies)."""
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


@pytest.mark.parametrize("N,M,kappa0", [(9, 10, 1.0), (8, 16, 1.0), (5, 10, 1.7), (4, 1, 0.6)])
def test_one_rounding_at_the_size_of_the_result(E, N, M, kappa0):
    s, sigma, T = 96, 0.002, np.longdouble
    kl, xi = E.kl_build(N, M), draw_xi(31, s, M)
    lo, hi = (t.cpu().numpy() for t in E.kl_extrema(N, kl, torch.as_tensor(xi, device=DEV), M, sigma, kappa0=kappa0))
    raw = kl.cpu().numpy()
    sq = raw[:8 * M].view(np.float64)
    tr = raw[44 * M:56 * M].view(np.int32).reshape(M, 3)
    off = (56 * M + 15) // 16 * 16
    phi = raw[off:off + 16 * M * N].view(np.float64).reshape(M, 2 * N).astype(T)
    modes = np.stack([np.einsum("z,y,x->zyx", phi[t[2]], phi[t[1]], phi[t[0]]).ravel() for t in tr])
    c = T(sigma) * sq.astype(T) * xi.astype(T)
    k = T(kappa0) + c @ modes
    mag = (np.abs(c) @ np.abs(modes)).max(1)
    for got, want in ((lo, k.min(1)), (hi, k.max(1))):
        err = np.abs(got.astype(T) - want)
        assert (err <= 2.0 ** -53 * (np.abs(want) + 40 * mag)).all(), float((err / np.abs(want)).max() * 2 ** 53)
