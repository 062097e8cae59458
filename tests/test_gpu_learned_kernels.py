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


# batches at the edges of the weight gradients' chunks (eight of 32 rows in
# flight) and of the bias sums' (sixteen of 16): one chunk, a partial group, a
# whole one, one past it.  Tolerances as in the network's parity test: the
# reference is FP64 on the same BF16 operands, and a pre-activation may round
# to the neighbouring BF16 value.
@pytest.mark.parametrize("B", [32, 96, 224, 256, 288, 544])
def test_network_batches(E, B):
    import numpy as np
    from oracle import learned as L
    rng = np.random.default_rng(B)
    p = L.init_params(12).astype(np.float32)
    X = rng.uniform(-1, 1, (B, L.IN)).astype(np.float32)
    T = rng.standard_normal((B, L.OUT)).astype(np.float32)
    dev = lambda a: torch.as_tensor(a, device=DEV)  # noqa: E731
    y, g, loss = E.mlp_grad(dev(p), dev(X), dev(T))
    yo, lo, go = L.forward_backward(p.astype(np.float64), X, T, bf16_points=True)
    rel = lambda a, b: np.linalg.norm(a - b) / np.linalg.norm(b)  # noqa: E731
    assert rel(y.cpu().numpy(), yo) <= 5e-3 and abs(float(loss.item()) - lo) <= 5e-3 * lo
    off, gg = 0, g.cpu().numpy()
    for name, shape in L.SIZES:
        k = int(np.prod(shape))
        assert rel(gg[off:off + k], go[off:off + k]) <= 2e-2, name
        off += k
    assert torch.equal(E.mlp_forward(dev(p), dev(X)), y)
    # the training step takes Adam on those gradients, bit for bit, the rows
    # in the order of its index list
    perm = rng.permutation(B).astype(np.int32)
    inv = np.argsort(perm)
    a, am, av = dev(p), torch.zeros(L.P, device=DEV), torch.zeros(L.P, device=DEV)
    lt = torch.zeros(1, device=DEV)
    E.mlp_train(a, am, av, 0, dev(X[inv]), dev(T[inv]), B, dev(perm), 1e-3, loss=lt)
    b, bm, bv = dev(p), torch.zeros(L.P, device=DEV), torch.zeros(L.P, device=DEV)
    E.mlp_adam(b, g, bm, bv, 1, 1e-3)
    assert torch.equal(a, b) and torch.equal(am, bm) and torch.equal(av, bv) and torch.equal(lt, loss)


def _abs_product_bound(a, b, terms):
    """Elementwise bound on two FP64 evaluations of a @ b."""
    return 2 * (terms + 2) * EPS * (a.abs() @ b.abs())


# the 128-row blocks of the symmetric product: one block whole and ragged, one
# past it, several; K below one range, ragged and split
@pytest.mark.parametrize("n,m", [(1, 1), (7, 3), (31, 128), (500, 129), (2000, 96), (700, 300), (9000, 257)])
def test_gram(E, n, m):
    S = _rand((n, m), n + m)
    G = E.pod_gram(S)
    assert bool(((G - S.t() @ S).abs() <= _abs_product_bound(S.t(), S, n)).all())
    assert torch.equal(G, G.t().contiguous())


# narrow, middle and wide right operands (the three tile widths and one past
# each), ragged rows and K
@pytest.mark.parametrize("n,m,r", [(1, 4, 4), (300, 40, 33), (129, 70, 64), (1000, 130, 65), (513, 200, 129),
                                   (40, 32, 32), (5000, 96, 16)])
def test_basis_and_projection_products(E, n, m, r):
    S, V, lam = _rand((n, m), 5), _rand((m, r), 6), _rand(r, 7).abs() + 0.5
    Phi = E.pod_basis(S, V, lam)
    ref, b = (S @ V) / lam.sqrt(), _abs_product_bound(S, V, m + 4) / lam.sqrt()
    sign = torch.sign(Phi.gather(0, Phi.abs().argmax(0)[None, :]))
    assert bool((sign > 0).all())
    flip = torch.sign((ref * Phi).sum(0))
    assert bool(((Phi - flip * ref).abs() <= b).all())
    C = E.pod_project(Phi, S)
    assert bool(((C - S.t() @ Phi).abs() <= _abs_product_bound(S.t(), Phi, n)).all())


# panels of 16 columns whole and ragged, one panel and many, few rows, rows past
# a workgroup's; spectra that fall slowly, fast enough that the first power
# step's columns are dependent to 1e-2 of their length or to rounding, and with
# exact zeros; k on both sides of what the rotations and the
# Cholesky factor of all columns keep in LDS, and odd.
# Columns orthonormal to 64 k roundings; eigenpair residuals and eigenvalues
# to m k roundings of the largest eigenvalue where the iteration has converged.
@pytest.mark.parametrize("m,k,r,ratio,rank", [
    (1, 1, 1, 2.0, 1), (5, 3, 2, 30.0, 5), (96, 48, 16, 2.25, 96), (300, 64, 32, 3.0, 300), (200, 97, 40, 1.3, 200),
    (200, 96, 40, 1.3, 200), (140, 65, 30, 1.4, 140), (2050, 64, 32, 1.3, 2050),
    (300, 64, 32, 1.5, 20), (700, 33, 20, 1.6, 700), (40, 16, 16, 1e3, 40), (300, 256, 64, 1.2, 300),
    (16, 16, 16, 10.0, 1)])
def test_eigenpairs(E, m, k, r, ratio, rank):
    Q, _ = torch.linalg.qr(_rand((m, m), m + k).cpu())
    lam = ratio ** -torch.arange(m, dtype=torch.float64)
    lam[rank:] = 0.0
    G = (Q * lam) @ Q.t()
    G = ((G + G.t()) / 2).to(DEV)
    V, l = E.pod_eig(G, r, _rand((m, k), 9), 12)
    eye = torch.eye(r, dtype=torch.float64, device=DEV)
    assert float((V.t() @ V - eye).abs().max()) <= 64 * k * EPS
    assert float((G @ V - V * l).norm()) <= 8 * m * k * EPS
    assert float((l.cpu() - lam[:r]).abs().max()) <= 8 * m * k * EPS
    assert bool((l[:-1] >= l[1:]).all())


@pytest.mark.parametrize("m,r", [(1, 1), (7, 5), (130, 32), (100, 1024), (2049, 33)])
def test_standardize(E, m, r):
    C = _rand((m, r), 3) * torch.arange(1, r + 1, device=DEV)
    mag = C.abs().mean(0) + C.abs().amax(0)
    for common in (False, True):
        mu, sd, T = E.pod_standardize(C, common=common)
        mean, dev = C.mean(0), C.std(0, unbiased=False)
        assert bool(((mu - mean).abs() <= 2 * (m + 2) * EPS * mag).all())
        want = dev.max().expand(r) if common else dev
        want = torch.where(want > 0, want, torch.ones_like(want))
        assert bool(((sd - want).abs() <= 4 * (m + 4) * EPS * mag.max()).all())
        assert bool(((T.double() - (C - mu) / sd).abs() <= 2.0 ** -24 * ((C - mu) / sd).abs() + 1e-300).all())
