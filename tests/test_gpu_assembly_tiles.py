"""The tiled assemblies at the sizes where their tiles end: meshes from one
element up (rows without an interior neighbour, tiles cut along each axis),
every ensemble size, and mode counts from none to the largest, whose x indices
need more than one pass of the column sums.  An entry is a sum of fewer than
200 products of magnitudes bounded by the matrix's largest entry or the
coefficient's terms, so FP64 differs from the oracle's order by less than
400 x 2^-53 < 1e-13 of the largest entry."""
import numpy as np
import pytest
import torch

from workloads import draw_vector, draw_xi

pytestmark = pytest.mark.gpu
DEV = "cuda"
VEL = (0.6, -0.3, 0.74)


@pytest.fixture(scope="module")
def E():
    from paper_1511_03703_amd import ens
    ens.lib()
    return ens


def _close(got, want):
    got = got.cpu().numpy()
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= 1e-13 * max(np.abs(want).max(), 1e-300)


@pytest.mark.parametrize("M", [0, 1, 5, 16])
@pytest.mark.parametrize("N,s", [(1, 4), (2, 8), (3, 32), (4, 16), (5, 4), (7, 32), (8, 8), (11, 16)])
def test_assemblies_at_the_ends_of_their_tiles(E, orc, N, s, M):
    sigma, alpha, beta, f = 0.05, 5.0, 30.0, 0.7
    xi = draw_xi(5200 + N, s, M) if M else np.zeros((s, 0))
    xt = torch.as_tensor(xi, device=DEV)
    g, kl = E.graph_build(N), E.kl_build(N, max(M, 1))
    rp, ci = orc.graph(N)
    v, v32, b = E.assemble(g, kl, xt, M, sigma, f=f, want32=True)
    vo, bo = orc.assemble_ensemble(N, rp, ci, M, 1.0, 1.0, sigma, f, xi)
    _close(v, vo)
    _close(b, bo)
    assert torch.equal(v32, v.float())
    # the matrix is symmetric to the last bit
    n = len(rp) - 1
    row = np.repeat(np.arange(n), np.diff(rp))
    order = np.lexsort((row, ci))  # the transpose's entries in this one's order
    assert torch.equal(v, v[torch.as_tensor(order, device=DEV)])

    u = draw_vector(5300 + N, (n, s), -0.05, 0.1)
    prob = E.nl_problem(M, sigma, alpha, beta, VEL, f=f)
    F, J, ld, J32 = E.nl_assemble(g, kl, xt, prob, torch.as_tensor(u, device=DEV), want_load=True, want_jac32=True)
    Fo, Jo, lo = orc.ens_nl_assemble(N, rp, ci, M, 1.0, 1.0, sigma, f, alpha, np.array(VEL), beta, xi, u)
    _close(F, Fo)
    _close(J, Jo)
    _close(ld, lo)
    assert torch.equal(J32, J.float())
