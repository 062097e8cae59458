"""The learned guess's kernels at the edges of their tiles and at every side
of their dispatch rules, against FP64 torch.  Tolerances are elementwise
rounding bounds: a sum of k products formed in FP64 in any order differs from
another by at most 2 (k + 2) 2^-53 times the sum of the products' magnitudes."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"
EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def E():
    from paper_1511_03703_amd import ens
    ens.lib()
    return ens


def _rand(shape, seed, dtype=torch.float64):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(shape, generator=g, dtype=torch.float64).to(dtype).to(DEV)


# r a multiple of 8 or not, whole and ragged chunks of 32, the largest r of
# the matrix-core form and the next; s below, at and past its tiles; n at the
# edges of the 16-row tiles and 64-row blocks; Phi off 16-byte alignment
@pytest.mark.parametrize("n,r,s,shift", [
    (1, 8, 8, 0), (15, 32, 32, 0), (16, 32, 33, 0), (65, 40, 9, 0), (1000, 24, 17, 0), (300, 256, 32, 0),
    (300, 264, 16, 0), (333, 7, 5, 0), (64, 32, 7, 0), (200, 32, 32, 1), (70000, 32, 64, 0)])
def test_reconstruct(E, n, r, s, shift):
    Phi = _rand(n * r + shift, 1)[shift:].view(n, r)
    c = _rand((s, r), 2, torch.float32)
    mu, sd = _rand(r, 3), _rand(r, 4)
    for m, d in ((mu, sd), (None, None), (mu, None)):
        x0 = E.pod_reconstruct(Phi, c, m, d)
        ch = c.double()
        if d is not None:
            ch = ch * d
        if m is not None:
            ch = ch + m
        bound = 2 * (r + 4) * EPS * (Phi.abs() @ (c.double().abs() * (1 if d is None else d.abs())
                                                  + (0 if m is None else m.abs())).t())
        assert bool(((x0 - Phi @ ch.t()).abs() <= bound).all())
