"""The ensemble products with their rows shared by several lane groups: every
ensemble size and precision, rows of every length from empty up, tiles whose
indices fit LDS and tiles whose do not, matrices below and above the size from
which wide ensembles take fewer groups, and the smallest systems.  A sum of k
products in any order differs from FP64's by at most (k + 2) roundings of the
sum of their magnitudes, plus the rounding of the result."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def E():
    from paper_1511_03703_amd import ens
    ens.lib()
    return ens


def _graph(E, lengths, n_cols, seed):
    g = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = np.concatenate([np.sort(g.choice(n_cols, k, replace=False)) for k in lengths] or [[]]).astype(np.int32)
    return E.graph_from_arrays(torch.as_tensor(rp, device=DEV), torch.as_tensor(ci, device=DEV))


def _check(E, g, s, dt, seed):
    gen = torch.Generator().manual_seed(seed)
    v = torch.randn((g.nnz, s), generator=gen, dtype=torch.float64).to(dt).to(DEV)
    x = torch.randn((g.n, s), generator=gen, dtype=torch.float64).to(dt).to(DEV)
    y = E.spmv(g, v, x)
    row = torch.repeat_interleave(torch.arange(g.n, device=DEV), (g.row_ptr[1:] - g.row_ptr[:-1]).long())
    t = v.double() * x.double()[g.col_idx.long()]
    ref = torch.zeros((g.n, s), dtype=torch.float64, device=DEV).index_add_(0, row, t)
    mag = torch.zeros_like(ref).index_add_(0, row, t.abs())
    k = float((g.row_ptr[1:] - g.row_ptr[:-1]).max())
    eps = 2.0 ** (-53 if dt == torch.float64 else -24)
    assert bool(((y.double() - ref).abs() <= (k + 3) * eps * mag).all())


@pytest.mark.parametrize("dt", [torch.float64, torch.float32])
@pytest.mark.parametrize("s", [4, 8, 16, 32])
def test_products_of_ragged_rows(E, s, dt):
    g = np.random.default_rng(s)
    # lengths 0 .. 31 (staged tiles), then rows too long for a tile's LDS
    for n, lengths in ((257, g.integers(0, 32, 257)), (130, g.integers(40, 90, 130)), (1, np.array([1]))):
        _check(E, _graph(E, lengths, n, s + n), s, dt, s)


# 256 MB of values lie between the first pairs of meshes for s = 32 in FP64 and
# FP32; 16 MB of gathered vector, up to which tiles go to an XCD in runs (of which
# the last is ragged), between the last two pairs
@pytest.mark.parametrize("N,s,dt", [(33, 32, torch.float64), (34, 32, torch.float64), (42, 32, torch.float32),
                                    (43, 32, torch.float32), (5, 4, torch.float32), (42, 16, torch.float64),
                                    (39, 32, torch.float64), (40, 32, torch.float64), (49, 32, torch.float32),
                                    (50, 32, torch.float32)])
def test_products_on_either_side_of_the_cache_size(E, N, s, dt):
    _check(E, E.graph_build(N), s, dt, N)


@pytest.mark.parametrize("s", [4, 8, 16, 32])
@pytest.mark.parametrize("n", [1, 2, 3, 9])
def test_solves_of_the_smallest_systems(E, s, n):
    # diagonally dominant symmetric tridiagonal systems, FP64 and refined
    lengths = np.array([min(i + 2, n) - max(i - 1, 0) for i in range(n)])
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = np.concatenate([np.arange(max(i - 1, 0), min(i + 2, n)) for i in range(n)]).astype(np.int32)
    g = E.graph_from_arrays(torch.as_tensor(rp, device=DEV), torch.as_tensor(ci, device=DEV))
    row = np.repeat(np.arange(n), lengths)
    scale = np.random.default_rng(n).uniform(1.0, 2.0, s)
    v = np.where(row == ci, 3.0, -1.0)[:, None] * scale[None, :]
    A = np.zeros((s, n, n))
    A[:, row, ci] = v.T
    b = np.random.default_rng(s).standard_normal((n, s))
    want = np.linalg.solve(A, b.T[:, :, None])[:, :, 0].T
    vt, bt = torch.as_tensor(v, device=DEV), torch.as_tensor(b, device=DEV)
    for kw in (dict(), dict(values32=vt.float())):
        x, st, rc = E.cg(g, vt, bt, opts=E.cg_opts(rtol=1e-12, mixed=bool(kw)), **kw)
        assert rc == E.ENS_OK, st
        # |x - x*| <= |A^-1| |r|, |A^-1| <= 1, |b| <= 5 |x*|
        assert np.linalg.norm(x.cpu().numpy() - want) <= 1e-11 * np.linalg.norm(b)
