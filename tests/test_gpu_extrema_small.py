"""The extremes of the coefficient on both sides of the bounds up to which a
sample has one workgroup (16^3, and 2048 samples): extremes are exact in any
order, so a few samples alone and among many give bitwise the same, with the
whole coefficient in FP64 within its roundings, and a sample that is not a number
has NaN for both."""
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


@pytest.mark.parametrize("N", [1, 2, 8, 9, 16, 17, 24])
@pytest.mark.parametrize("M", [0, 1, 10])
def test_one_workgroup_a_sample_and_many(E, N, M):
    s, sigma = 2100, 0.2
    kl, xi = E.kl_build(N, M), draw_xi(7, s, max(M, 1))[:, :M].copy()
    if M:
        xi[2, M - 1] = np.nan
        xi[s - 1, 0] = np.nan
    t = torch.as_tensor(xi, device=DEV)
    many = [v.cpu().numpy() for v in E.kl_extrema(N, kl, t, M, sigma)]
    few = [v.cpu().numpy() for v in E.kl_extrema(N, kl, t[:5].contiguous(), M, sigma)]
    for a, b in zip(many, few):
        assert np.array_equal(a[:5], b, equal_nan=True)
    bad = np.isnan(xi).any(1) if M else np.zeros(s, bool)
    assert np.array_equal(np.isnan(many[0]), bad) and np.array_equal(np.isnan(many[1]), bad)
    k = np.ones((s, 1))
    mag = np.ones(s)
    if M:
        raw = kl.cpu().numpy()
        sq, tr = raw[:8 * M].view(np.float64), raw[44 * M:56 * M].view(np.int32).reshape(M, 3)
        off = (56 * M + 15) // 16 * 16
        phi = raw[off:off + 16 * M * N].view(np.float64).reshape(M, 2 * N)
        modes = np.stack([np.einsum("z,y,x->zyx", phi[q[2]], phi[q[1]], phi[q[0]]).ravel() for q in tr])
        c = sigma * sq * xi[:40]
        k, mag = 1.0 + c @ modes, 1.0 + (np.abs(c) @ np.abs(modes)).max(1)
    ok = ~bad[:len(k)]
    # both sums: M + 3 roundings of the magnitudes, and the table's mirror images
    tol = 2.0 ** -53 * (2 * M + 46) * mag
    assert (np.abs(many[0][:len(k)] - k.min(1))[ok] <= tol[:len(k)][ok]).all()
    assert (np.abs(many[1][:len(k)] - k.max(1))[ok] <= tol[:len(k)][ok]).all()
