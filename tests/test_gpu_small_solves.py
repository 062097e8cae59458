"""The CG iteration of small FP64 systems, whose kernels hold the reductions
before them: sizes on both sides of the smallest and the largest system that
takes it and of the partial rows that need a stage of their own, one workgroup
and many, coupled and compacted solves, and polls at every distance.

The systems are symmetric tridiagonal with eigenvalues of at least d - 2 and at
most d + 2, d from 2.5 to 4, so |x - x*| <= |r| / 0.5 and |b| <= 6 |x*|; a
residual below rtol |b| = 1e-11 |b| (and FP64's drift of the recursion, some
1e-15 |b| an iteration) bounds the error by 3e-11 |b| for each sample."""
import numpy as np
import pytest
import torch
from scipy.linalg import solve_banded

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def E():
    from paper_1511_03703_amd import ens
    ens.lib()
    return ens


def _system(E, n, s):
    rp = np.concatenate([[0], np.cumsum(np.full(n, 3))])
    ci = (np.arange(n)[:, None] + np.array([-1, 0, 1])[None, :]).ravel()
    keep = (ci >= 0) & (ci < n)
    rp = np.concatenate([[0], np.cumsum(keep)])[rp].astype(np.int32)
    row = np.repeat(np.arange(n), 3)[keep]
    ci = ci[keep].astype(np.int32)
    diag = np.linspace(2.5, 4.0, s)
    v = np.where((row == ci)[:, None], diag[None, :], -1.0)
    b = np.random.default_rng(n).standard_normal((n, s))
    g = E.graph_from_arrays(torch.as_tensor(rp, device=DEV), torch.as_tensor(ci, device=DEV))
    return g, torch.as_tensor(v, device=DEV), torch.as_tensor(b, device=DEV), diag, b


def _error(x, diag, b):
    n = len(b)
    x = x.cpu().numpy()
    err = []
    for e in range(b.shape[1]):
        ab = np.full((3, n), -1.0)
        ab[1] = diag[e]
        err.append(np.linalg.norm(x[:, e] - solve_banded((1, 1), ab, b[:, e])) / np.linalg.norm(b[:, e]))
    return max(err)


# the smallest of them has about 3700 values, the largest 2^21; partials fill
# 32 KB at 1024 s = 4 rows of one quantity and 128 s = 16 rows of two
@pytest.mark.parametrize("n,s", [(110, 32), (120, 32), (900, 4), (1000, 4), (257, 16), (4097, 8), (2048, 16), (16385, 4),
                                 (33001, 16), (2 ** 16, 32), (2 ** 16 + 1, 32), (2 ** 19, 4), (2 ** 19 + 1, 4)])
def test_solves_on_either_side_of_the_bounds(E, n, s):
    g, v, b, diag, bh = _system(E, n, s)
    x, st, rc = E.cg(g, v, b, opts=E.cg_opts(rtol=1e-11))
    assert rc == E.ENS_OK, st
    assert _error(x, diag, bh) <= 3e-11


@pytest.mark.parametrize("kw", [dict(check_every=1), dict(check_every=7), dict(check_every=1000), dict(coupled=True),
                                dict(compact=True, check_every=2)])
def test_options(E, kw):
    g, v, b, diag, bh = _system(E, 3000, 16)
    _, want, _ = E.cg(g, v, b, opts=E.cg_opts(rtol=1e-11, coupled=kw.get("coupled", False)))
    x, st, rc = E.cg(g, v, b, opts=E.cg_opts(rtol=1e-11, **kw))
    assert rc == E.ENS_OK, st
    # a coupled solve stops on the ensemble's norm: sqrt(s) of a sample's
    assert _error(x, diag, bh) <= 3e-11 * (5.0 if "coupled" in kw else 1.0)
    assert [a["iters"] for a in st] == [a["iters"] for a in want]


@pytest.mark.parametrize("n", [3000, 2 ** 18 + 1])
@pytest.mark.parametrize("check_every", [1, 5, 100])
def test_iteration_limit_and_the_iterates_before_it(E, n, check_every):
    g, v, b, diag, bh = _system(E, n, 8)
    x, st, rc = E.cg(g, v, b, opts=E.cg_opts(rtol=1e-11, max_iter=6, check_every=check_every))
    assert rc != E.ENS_OK and [a["iters"] for a in st] == [6] * 8
    # six steps of the recursion in NumPy: the same up to rounding
    for e in (0, 7):
        A = lambda p: diag[e] * p - np.concatenate([[0.0], p[:-1]]) - np.concatenate([p[1:], [0.0]])  # noqa: E731
        xr, r = np.zeros(n), bh[:, e].copy()
        p, rho = r / diag[e], r @ r / diag[e]
        for _ in range(6):
            q = A(p)
            alpha = rho / (p @ q)
            xr, r = xr + alpha * p, r - alpha * q
            rho, old = r @ r / diag[e], rho
            p = r / diag[e] + rho / old * p
        assert np.linalg.norm(x[:, e].cpu().numpy() - xr) <= 1e-12 * np.linalg.norm(bh[:, e])
