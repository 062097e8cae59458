"""The CG iteration of small FP64 systems at its lower bound: its second control
block (3376 bytes) lies at the end of the vector whose other half holds partial
sums, in systems whose vectors hold eight of it: 3376 values and more.  Sizes
one row and a tile's rows to either side for every ensemble size, warm and cold
starts, against a direct solve.

The systems are symmetric tridiagonal with eigenvalues of at least d - 2, d from
2.5 to 4, so |x - x*| <= |r| / 0.5; a residual below 1e-11 |b| (and FP64's drift
of the recursion, some 1e-15 |b| an iteration) bounds the error by 3e-11 |b|."""
import numpy as np
import pytest
import torch
from scipy.linalg import solve_banded

pytestmark = pytest.mark.gpu
DEV = "cuda"
VALUES = 3376


@pytest.fixture(scope="module")
def E():
    from paper_1511_03703_amd import ens
    ens.lib()
    return ens


def _sizes():
    for s in (4, 8, 16, 32):
        n = -(-VALUES // s)  # the first that takes the iteration
        for k in (n - 16, n - 1, n, n + 1, n + 16):
            yield k, s


@pytest.mark.parametrize("n,s", list(_sizes()))
@pytest.mark.parametrize("warm", [False, True])
def test_either_side_of_the_bound(E, n, s, warm):
    rp = np.minimum(np.maximum(3 * np.arange(n + 1) - 1, 0), 3 * n - 2).astype(np.int32)
    ci = (np.arange(n)[:, None] + np.array([-1, 0, 1])).ravel()
    row = np.repeat(np.arange(n), 3)
    keep = (ci >= 0) & (ci < n)
    ci, row = ci[keep].astype(np.int32), row[keep]
    diag = np.linspace(2.5, 4.0, s)
    v = np.where((row == ci)[:, None], diag, -1.0)
    rng = np.random.default_rng(n)
    b = rng.standard_normal((n, s))
    g = E.graph_from_arrays(torch.as_tensor(rp, device=DEV), torch.as_tensor(ci, device=DEV))
    x0 = torch.as_tensor(rng.standard_normal((n, s)) if warm else np.zeros((n, s)), device=DEV)
    opts = E.cg_opts(rtol=1e-11)
    # a workspace of exactly the bytes asked for, a pattern behind it
    need = E.cg_workspace_bytes(g, s, opts)
    buf = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device=DEV)
    x, st, rc = E.cg(g, torch.as_tensor(v, device=DEV), torch.as_tensor(b, device=DEV), x=x0, opts=opts,
                     workspace=buf[:need])
    assert rc == E.ENS_OK, st
    assert bool((buf[need:] == 0x5A).all())
    x = x.cpu().numpy()
    for e in range(s):
        ab = np.full((3, n), -1.0)
        ab[1] = diag[e]
        assert np.linalg.norm(x[:, e] - solve_banded((1, 1), ab, b[:, e])) <= 3e-11 * np.linalg.norm(b[:, e])
