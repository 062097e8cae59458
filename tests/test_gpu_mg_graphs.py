"""Multigrid CG on a fine graph with fewer stored entries than the mesh's full
27-point pattern.

The face neighbours' entries of an assembled matrix (small beside the others)
are lumped onto the diagonal, once as stored zeros of the full graph and once
with those entries and the boundary's zeros left out.  Both are the same
symmetric M-matrix, so both solves take the same iterations (one more or less:
their products round differently) to the same solution: with A x = b and
|r| <= 1e-10 |b| on each side the two differ by at most 2e-10 |b| / lmin(A), and
lmin = 3 pi^2 kappa_min h^3 (1 + O(h^2)) on the interior, |b| = h^3 sqrt(n), for
kappa >= 0.5 here.  The full matrix is larger than the 256 MB from which the row
passes change their tiles, the other one smaller."""
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


def _lumped(g, v):
    """Values with the face entries of interior rows moved to the diagonal, and
    which entries are then needed."""
    n1 = g.N + 1
    row = torch.repeat_interleave(torch.arange(g.n, device=DEV), (g.row_ptr[1:] - g.row_ptr[:-1]).long())
    d = g.col_idx.long() - row
    face = (d.abs() == 1) | (d.abs() == n1) | (d.abs() == n1 * n1)
    diag = torch.nonzero(d == 0).ravel()
    out = v.clone()
    out[diag] += torch.zeros_like(v[:g.n]).index_add_(0, row, v * face[:, None])
    out[face] = 0.0
    return out, (out != 0.0).any(1)


@pytest.mark.parametrize("galerkin", [False, True])
def test_fewer_entries_than_the_mesh(E, galerkin):
    N, s, M, sigma = 36, 32, 3, 0.2
    g, kl = E.graph_build(N), E.kl_build(N, M)
    xi = torch.as_tensor(draw_xi(77, s, M), device=DEV)
    v, _, b = E.assemble(g, kl, xi, M, sigma)
    v, need = _lumped(g, v)
    counts = torch.zeros(g.n, dtype=torch.int64, device=DEV)
    row = torch.repeat_interleave(torch.arange(g.n, device=DEV), (g.row_ptr[1:] - g.row_ptr[:-1]).long())
    counts.index_add_(0, row, need.long())
    rp = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), torch.cumsum(counts, 0)]).int()
    small = E.graph_from_arrays(rp.contiguous(), g.col_idx[need].contiguous(), N)
    vs = v[need].contiguous()
    assert small.nnz * s * 8 <= 256 << 20 < g.nnz * s * 8
    mg = E.Multigrid(N, M, s)
    opts = E.cg_opts(rtol=1e-10, check_every=4)
    if galerkin:
        mg.setup_galerkin(g, v)
    else:
        mg.setup(g, v, xi, sigma)
    x, st, rc = E.cg_mg(g, v, b, mg, opts=opts)
    assert rc == E.ENS_OK, st
    if not galerkin:
        mg.setup(small, vs, xi, sigma)
    xs, ss, rc = E.cg_mg(small, vs, b, mg, opts=opts)
    assert rc == E.ENS_OK, ss
    print([t["iters"] for t in st], [t["iters"] for t in ss])
    assert all(abs(p["iters"] - q["iters"]) <= 1 for p, q in zip(st, ss))
    bound = 2e-10 * np.sqrt(g.n) / (3 * np.pi ** 2 * 0.5)
    assert float((x - xs).norm(dim=0).max()) <= bound
