"""Performance cases: the work a program has this framework do, through the
public entry points of ``paper_1511_03703_amd``.

``listed()`` names the cases, ``draw(rng)`` draws one more of the same ranges,
``prepare`` makes what a program holds before the call (inputs from the seed,
graph, KL table, hierarchy, workspace), ``run`` is one pass, ``work`` the bytes
and operations a pass cannot do without, and ``exact`` the same outputs in
plain 64-bit torch.

Kinds of work:

solve     assembly of an ensemble and its CG solve (Jacobi, or multigrid with
          the set-up of its hierarchy in the pass, in FP64 or FP32 inside FP64
          refinement)
newton    the nonlinear problem: the preconditioner's matrices and Newton with
          multigrid-preconditioned GMRES
batch     sample groups on meshes of several sizes through the resident pool
spmv      the ensemble sparse product
contrast  the grouping predictor: each sample's coefficient contrast, and the
          order of the samples by it
basis     the POD basis and network targets from solved snapshots
train     Adam steps of the network on mini-batches
guess     the trained network's initial guess lifted to the mesh
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1511_03703_amd import batchpool, ens
from paper_1511_03703_amd.learned import LearnedGuess

DEV = "cuda"
VEL = (3 ** -0.5, 3 ** -0.5, 3 ** -0.5)

# meshes whose hierarchy ends in a small coarsest level
MG_MESHES = (8, 10, 12, 14, 16, 18, 20, 24, 28, 32, 36, 40, 48, 56, 64, 72, 80, 96, 112, 128)


# ------------------------------------------------------------------- cases


def listed():
    return [
        # the smallest solve in use (parity checks, interactive exploration):
        # 35 iterations on vectors of 20,000 values, where latency counts
        dict(name="solve_16_s4", kind="solve", N=16, s=4, M=3, sigma=0.1, rtol=1e-10, precond="jacobi", mixed=False),
        # an odd mesh, which no hierarchy fits, at a small ensemble
        dict(name="solve_37_s8", kind="solve", N=37, s=8, M=10, sigma=0.2, rtol=1e-10, precond="jacobi", mixed=False),
        # the ordinary FP64 solve: one ensemble on a middling mesh
        dict(name="solve_64_s16_mg", kind="solve", N=64, s=16, M=10, sigma=0.2, rtol=1e-10, precond="mg",
             mixed=False),
        # the headline solve: FP32 multigrid CG inside FP64 refinement
        dict(name="solve_128_s32_mixed", kind="solve", N=128, s=32, M=10, sigma=0.3, rtol=1e-8, precond="mg",
             mixed=True),
        # the nonlinear problem with advection and reaction
        dict(name="newton_64_s16", kind="newton", N=64, s=16, M=10, sigma=0.3, alpha=10.0, beta=100.0, rtol=1e-8),
        # a wave of groups on every mesh of the batch workload
        dict(name="batch_8x16", kind="batch", meshes="32,48,64,96,48,32,64,48", s=16, M=10, sigma=0.2, rtol=1e-8),
        # the ensemble product itself: a large FP32 one (the refinement's), and
        # a small FP64 one of odd size at a narrow ensemble
        dict(name="spmv_96_s32_f32", kind="spmv", N=96, s=32, M=10, sigma=0.3, fp64=False),
        dict(name="spmv_27_s8_f64", kind="spmv", N=27, s=8, M=10, sigma=0.2, fp64=True),
        # the samples of a batch's 64^3 groups ranked before they are grouped
        dict(name="contrast_64_512", kind="contrast", N=64, samples=512, M=10, sigma=0.2),
        # the learned guess: its basis from 2048 snapshots, an epoch and a half
        # of the network's training, and the guess that each solve starts from
        dict(name="basis_64_2048", kind="basis", N=64, m=2048),
        dict(name="train_256x64", kind="train", count=2048, batch=256, steps=64),
        dict(name="guess_64_s32", kind="guess", N=64, s=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("solve", "solve", "solve", "solve", "newton", "batch", "spmv", "spmv", "contrast", "basis",
                       "train", "guess"))
    M = rng.randint(3, 10)
    sigma = round(rng.uniform(0.1, 0.3), 3)
    s = rng.choice((4, 8, 16, 32))
    if kind == "solve":
        if rng.random() < 0.5:
            return dict(kind=kind, N=_log_int(rng, 8, 72), s=s, M=M, sigma=sigma, rtol=1e-10, precond="jacobi",
                        mixed=False)
        mixed = rng.random() < 0.5
        return dict(kind=kind, N=rng.choice(MG_MESHES), s=s, M=M, sigma=sigma, rtol=1e-8 if mixed else 1e-10,
                    precond="mg", mixed=mixed)
    if kind == "newton":
        return dict(kind=kind, N=rng.choice([N for N in MG_MESHES if 16 <= N <= 64]), s=s, M=M, sigma=sigma,
                    alpha=round(rng.uniform(2.0, 10.0), 2), beta=round(rng.uniform(10.0, 100.0), 1), rtol=1e-8)
    if kind == "batch":
        meshes = [rng.choice((16, 24, 31, 32, 40, 48, 57, 64)) for _ in range(rng.randint(2, 8))]
        return dict(kind=kind, meshes=",".join(str(N) for N in meshes), s=rng.choice((8, 16)), M=M, sigma=sigma,
                    rtol=1e-8)
    if kind == "spmv":
        return dict(kind=kind, N=_log_int(rng, 8, 112), s=s, M=M, sigma=sigma, fp64=rng.random() < 0.5)
    if kind == "contrast":
        return dict(kind=kind, N=_log_int(rng, 16, 96), samples=_log_int(rng, 32, 1024), M=M, sigma=sigma)
    if kind == "basis":
        return dict(kind=kind, N=_log_int(rng, 12, 64), m=32 * _log_int(rng, 4, 56))
    if kind == "train":
        return dict(kind=kind, count=_log_int(rng, 256, 4096), batch=32 * _log_int(rng, 1, 32),
                    steps=_log_int(rng, 16, 96))
    return dict(kind=kind, N=_log_int(rng, 8, 96), s=32 * rng.randint(1, 2))


# ----------------------------------------------------------------- inputs


def _xi(seed, count, M):
    """KL inputs y ~ U[-1, 1]^M, one row per sample."""
    return np.random.default_rng(seed).uniform(-1.0, 1.0, (count, M))


def _modes(N, count, seed):
    """`count` smooth orthonormal fields [n][count], zero on the boundary:
    random combinations of products of sines (no symmetry of the cube)."""
    g = np.random.default_rng(seed)
    K = 7
    t = torch.linspace(0.0, 1.0, N + 1, dtype=torch.float64, device=DEV)
    sn = torch.sin(math.pi * torch.arange(1, K + 1, dtype=torch.float64, device=DEV)[:, None] * t[None, :])
    sn[:, 0] = 0.0
    sn[:, -1] = 0.0
    w = g.standard_normal((count, K, K, K))
    a = np.arange(1, K + 1)
    w /= (a[:, None, None] ** 2 + a[None, :, None] ** 2 + a[None, None, :] ** 2)
    w = torch.as_tensor(w, device=DEV)
    f = (w.reshape(count * K * K, K) @ sn).reshape(count * K, K, N + 1)           # [c kz][ky][x]
    f = (sn.t() @ f.transpose(0, 1).reshape(K, -1)).reshape(N + 1, count, K, N + 1)  # [y][c][kz][x]
    f = f.permute(2, 0, 1, 3).reshape(K, -1)
    f = (sn.t() @ f).reshape(N + 1, N + 1, count, N + 1)                          # [z][y][c][x]
    f = f.permute(0, 1, 3, 2).reshape(-1, count).contiguous()                     # [n][count], x fastest
    for _ in range(2):
        c = torch.linalg.cholesky((f.t() @ f).cpu())
        f = f @ torch.linalg.inv(c).t().to(DEV)
    return f.contiguous()


def _snapshots(N, m, seed):
    """m snapshots [n][m] like solutions: a mean field, then modes of falling
    weight."""
    count = min(m, 96, (N - 1) ** 3)
    q = _modes(N, count, seed)
    g = np.random.default_rng(seed + 1)
    z = g.standard_normal((count, m)) * (0.05 * 0.9 ** np.arange(count))[:, None]
    z[0] = 1.0 + 0.1 * g.standard_normal(m)
    return (q @ torch.as_tensor(z, device=DEV)).contiguous()


def _targets(xi, seed):
    """Smooth network targets [count][32] of the inputs, later ones smaller."""
    g = np.random.default_rng(seed)
    lin = g.standard_normal((xi.shape[1], 32))
    quad = 0.3 * g.standard_normal((xi.shape[1], 32))
    return ((xi @ lin + (xi * xi) @ quad) * 0.85 ** np.arange(32)).astype(np.float32)


class _State:
    pass


def prepare(case, seed):
    st = _State()
    st.case = case
    kind = case["kind"]
    if kind in ("solve", "newton", "spmv"):
        N, s, M = case["N"], case["s"], case["M"]
        st.g = ens.graph_build(N, device=DEV)
        st.kl = ens.kl_build(N, M, device=DEV)
        st.xi = torch.as_tensor(_xi(seed, s, M), device=DEV)
        g = st.g
        if kind == "spmv":
            vals, v32, _ = ens.assemble(g, st.kl, st.xi, M, case["sigma"], want32=not case["fp64"])
            st.vals = vals if case["fp64"] else v32
            x = torch.as_tensor(np.random.default_rng(seed + 1).uniform(-1.0, 1.0, (g.n, s)), device=DEV)
            st.x = x if case["fp64"] else x.float()
            st.y = torch.empty_like(st.x)
            return st
        st.rhs = torch.empty((g.n, s), dtype=torch.float64, device=DEV)
        st.u = torch.empty_like(st.rhs)
        if kind == "solve":
            mg, mixed = case["precond"] == "mg", case["mixed"]
            st.vals = torch.empty((g.nnz, s), dtype=torch.float64, device=DEV)
            st.vals32 = torch.empty((g.nnz, s), dtype=torch.float32, device=DEV) if mixed else None
            st.opts = ens.cg_opts(rtol=case["rtol"], mixed=mixed, inner_rtol=1e-4 if mg else 1e-5,
                                  check_every=4 if mg else 16)
            st.ws = torch.empty(ens.cg_workspace_bytes(g, s, st.opts), dtype=torch.uint8, device=DEV)
            st.mg = ens.Multigrid(N, M, s, fp32=mixed, device=DEV) if mg else None
            return st
        st.vals32 = torch.empty((g.nnz, s), dtype=torch.float32, device=DEV)
        st.prob = ens.nl_problem(M, case["sigma"], case["alpha"], case["beta"], VEL)
        st.mg = ens.Multigrid(N, M, s, fp32=True, device=DEV)
        st.opts = ens.newton_opts(rtol=case["rtol"], lin_rtol=0.3, restart=30, jac32=True, forcing=ens.FORCING_EW)
        st.ws = torch.empty(ens.newton_workspace_bytes(g, s, st.opts), dtype=torch.uint8, device=DEV)
        return st
    if kind == "batch":
        meshes, s = _meshes(case), case["s"]
        need = sum(batchpool.group_buffer_bytes(N, s) + batchpool.group_workspace_bound(N, s) for N in meshes)
        st.pool = batchpool.BatchPool(ens, meshes, s, case["M"], need + (1 << 20), device=DEV)
        st.xi = torch.as_tensor(_xi(seed, len(meshes) * s, case["M"]).reshape(len(meshes), s, -1), device=DEV)
        st.opts = ens.batch_opts(rtol=case["rtol"])
        return st
    if kind == "contrast":
        st.kl = ens.kl_build(case["N"], case["M"], device=DEV)
        st.xi = torch.as_tensor(_xi(seed, case["samples"], case["M"]), device=DEV)
        return st
    if kind == "basis":
        st.S = _snapshots(case["N"], case["m"], seed)
        return st
    if kind == "train":
        count, batch, steps = case["count"], case["batch"], case["steps"]
        xi = _xi(seed, count, ens.MLP_IN)
        st.xi = torch.as_tensor(xi.astype(np.float32), device=DEV)
        st.T = torch.as_tensor(_targets(xi, seed + 1), device=DEV)
        st.p0 = ens.mlp_init(seed + 2, DEV)
        st.idx = torch.as_tensor(_order(case, seed), device=DEV)
        return st
    st.lg = LearnedGuess(r=32, device=DEV)
    st.lg.Phi = _modes(case["N"], 32, seed)
    st.lg.mu, st.lg.sd = (torch.as_tensor(v, device=DEV) for v in _scales(seed))
    st.lg.params = ens.mlp_init(seed + 2, DEV)
    st.xi = torch.as_tensor(_xi(seed, case["s"], ens.MLP_IN).astype(np.float32), device=DEV)
    st.x0 = torch.empty((st.lg.Phi.shape[0], case["s"]), dtype=torch.float64, device=DEV)
    return st


def _meshes(case):
    return [int(v) for v in case["meshes"].split(",")]


def _order(case, seed):
    """Shuffled rows of the training set, one permutation after the other."""
    need = case["batch"] * case["steps"]
    g = np.random.default_rng(seed + 3)
    rows = [g.permutation(case["count"]) for _ in range(-(-need // case["count"]))]
    return np.concatenate(rows)[:need].astype(np.int32)


def _scales(seed):
    g = np.random.default_rng(seed + 1)
    mu = g.standard_normal(32) * 0.9 ** np.arange(32)
    return mu, np.full(32, 0.2)


# ------------------------------------------------------------------ a pass


def _iters(stats):
    return torch.tensor([t["iters"] for t in stats], dtype=torch.int64)


def run(st):
    case = st.case
    kind = case["kind"]
    if kind == "spmv":
        return ens.spmv(st.g, st.vals, st.x, y=st.y)
    if kind == "solve":
        if st.mg is not None:
            st.mg.assemble_setup(st.g, st.kl, st.xi, case["sigma"], st.vals, st.rhs, values32=st.vals32)
            st.u.zero_()
            x, stats, _ = ens.cg_mg(st.g, st.vals, st.rhs, st.mg, x=st.u, values32=st.vals32, opts=st.opts,
                                    workspace=st.ws)
        else:
            ens.assemble(st.g, st.kl, st.xi, case["M"], case["sigma"], values=st.vals, values32=st.vals32, rhs=st.rhs)
            st.u.zero_()
            x, stats, _ = ens.cg(st.g, st.vals, st.rhs, x=st.u, values32=st.vals32, opts=st.opts, workspace=st.ws)
        return dict(x=x, rhs=st.rhs, iters=_iters(stats))
    if kind == "newton":
        st.mg.assemble_setup_adv(st.g, st.kl, st.xi, st.prob, None, st.rhs, values32=st.vals32)
        st.u.zero_()
        u, stats, _ = ens.newton(st.g, st.kl, st.xi, st.prob, u=st.u, opts=st.opts, mg=st.mg, mg_values=st.vals32,
                                 workspace=st.ws)
        return dict(u=u, iters=torch.tensor([t["newton_iters"] for t in stats], dtype=torch.int64))
    if kind == "batch":
        xs = []

        def keep(wave, groups, stats):
            xs.extend(x.clone() for _, _, _, x in groups)

        stats, _ = st.pool.run(st.xi, case["sigma"], st.opts, on_wave=keep)
        return dict(x=xs, iters=[_iters(t) for t in stats])
    if kind == "contrast":
        kmin, kmax = ens.kl_extrema(case["N"], st.kl, st.xi, case["M"], case["sigma"])
        perm = ens.group_order((kmax / kmin).cpu().numpy())
        return dict(kmin=kmin, kmax=kmax, order=perm)
    if kind == "basis":
        lg = LearnedGuess(r=32, device=DEV)
        T = lg.fit_basis(st.S, eig_seed=7)
        return dict(T=T, Phi=lg.Phi, lam=lg.lam, mu=lg.mu, sd=lg.sd)
    if kind == "train":
        p = st.p0.clone()
        m, v = torch.zeros_like(p), torch.zeros_like(p)
        loss = torch.zeros(case["steps"], dtype=torch.float32, device=DEV)
        ens.mlp_train(p, m, v, 0, st.xi, st.T, case["batch"], st.idx, 1e-3, loss=loss)
        return dict(params=p, m=m, v=v, loss=loss)
    return st.lg.guess(st.xi, x0=st.x0)


# -------------------------------------------------------------------- work


def work(case):
    """A solve reads its matrix once per product its iterations make (one a
    CG iteration and, in a multigrid one, four on each level of the cycle,
    8/7 of the finest), at the iteration counts such problems take; the
    assembly writes it once.  Everything else: inputs read once, outputs
    written once."""
    kind = case["kind"]
    if kind in ("solve", "newton", "spmv"):
        n, nnz = (case["N"] + 1) ** 3, (3 * case["N"] + 1) ** 3
        s = case["s"]
        if kind == "spmv":
            w = 8 if case["fp64"] else 4
            return dict(bytes=nnz * (s * w + 4) + 4 * n + 2 * n * s * w, flops=2 * nnz * s)
        return dict(zip(("bytes", "flops"), _solve_work(case, n, nnz, s)))
    if kind == "batch":
        b = f = 0.0
        for N in _meshes(case):
            c = dict(case, kind="solve", N=N, precond="jacobi", mixed=False)
            bb, ff = _solve_work(c, (N + 1) ** 3, (3 * N + 1) ** 3, case["s"])
            b += bb
            f += ff
        return dict(bytes=b, flops=f)
    if kind == "contrast":
        # the coefficient at 8 N^3 points by axis-wise contraction
        pts = 8 * case["N"] ** 3
        return dict(bytes=8 * case["samples"] * (case["M"] + 2), flops=2 * case["M"] * pts * case["samples"])
    if kind == "basis":
        n, m, r = (case["N"] + 1) ** 3, case["m"], 32
        # half of the symmetric Gram, the basis, the projection
        return dict(bytes=8 * (n * m + n * r + m * r), flops=n * m * (m + 4 * r))
    if kind == "train":
        fl = 6 * (10 * 256 + 256 * 256 + 256 * 32) * case["batch"] * case["steps"]
        return dict(bytes=76832 * 4 * 7 + case["batch"] * case["steps"] * (4 + 4 * 42), flops=fl)
    n, s = (case["N"] + 1) ** 3, case["s"]
    return dict(bytes=8 * n * 32 + 8 * n * s + 4 * 76832, flops=2 * n * s * 32 + 2 * s * 76544)


def _solve_work(case, n, nnz, s):
    wide = nnz * (8 * s + 4)
    narrow = nnz * (4 * s + 4)
    if case["kind"] == "newton":
        # FP32 cycle and Jacobian: the matrices written, 4 Newton steps of
        # about 2 products and cycles each
        b = 5 * 4 * nnz * s + 8 * narrow * (1 + 4 * 8 / 7)
        return b, 8 * 2 * nnz * s * (1 + 4 * 8 / 7)
    if case["precond"] == "jacobi":
        it = 2.5 * case["N"] * (-math.log10(case["rtol"]) / 10)
        return 8 * nnz * s + it * (wide + 8 * 4 * n * s), it * 2 * nnz * s
    if case["mixed"]:
        it = 6
        return 12 * nnz * s + 2 * wide + it * narrow * (1 + 4 * 8 / 7), it * 2 * nnz * s * (1 + 4 * 8 / 7)
    it = 7.5
    return 8 * nnz * s + it * wide * (1 + 4 * 8 / 7), it * 2 * nnz * s * (1 + 4 * 8 / 7)


# ----------------------------------------------- the same in 64-bit torch


def _kl_modes(M):
    """1D eigenpairs of exp(-|t - t'|) on [0, 1] by bisection, and the first M
    3D modes by eigenvalue, ties by ascending index triple."""
    om, lam, norm = [], [], []
    for t in range(M):
        m, odd = t // 2 + 1, t & 1
        lo, hi = ((m - 0.5), m) if odd else ((m - 1), (m - 0.5))
        lo, hi = 2 * math.pi * lo, 2 * math.pi * hi

        def eq(w):
            return w * math.cos(w / 2) + math.sin(w / 2) if odd else math.cos(w / 2) - w * math.sin(w / 2)

        flo = eq(lo)
        for _ in range(200):
            mid = 0.5 * (lo + hi)
            if (eq(mid) < 0) == (flo < 0):
                lo = mid
            else:
                hi = mid
        w = 0.5 * (lo + hi)
        om.append(w)
        lam.append(2.0 / (w * w + 1.0))
        s2 = math.sin(w) / (2 * w)
        norm.append(1.0 / math.sqrt(0.5 - s2 if odd else 0.5 + s2))
    triples = []
    for i in range(M):
        for j in range(M):
            for k in range(M):
                a, b, c = sorted((i, j, k))
                triples.append((-((lam[a] * lam[b]) * lam[c]), i, j, k))
    triples.sort()
    return om, norm, [(math.sqrt(-p), (i, j, k)) for p, i, j, k in triples[:M]]


def _gauss():
    r = 1.0 / math.sqrt(3.0)
    return 0.5 * (1.0 - r), 0.5 * (1.0 + r)


class _Kappa:
    """kappa at Gauss point q of every element: [z][y][x][sample]."""

    def __init__(self, N, M, sigma, xi):
        self.N, self.sigma = N, sigma
        om, norm, self.modes = _kl_modes(M)
        self.xi = torch.as_tensor(xi, device=DEV)
        pts = [(torch.arange(N, dtype=torch.float64, device=DEV) + g) / N - 0.5 for g in _gauss()]
        self.phi = [[norm[k] * (torch.sin(om[k] * p) if k & 1 else torch.cos(om[k] * p)) for p in pts]
                    for k in range(M)]

    def at(self, qz, qy, qx):
        N, M = self.N, len(self.modes)
        zy = torch.stack([(self.phi[t[2]][qz][:, None] * self.phi[t[1]][qy][None, :]).reshape(-1)
                          for _, t in self.modes], 1)
        xs = torch.stack([self.phi[t[0]][qx][:, None] * (self.sigma * sq * self.xi[:, m])[None, :]
                          for m, (sq, t) in enumerate(self.modes)], 0).reshape(M, -1)
        return (1.0 + zy @ xs).reshape(N, N, N, -1)


def _shapes():
    """Values [q][a] and unit-cube gradients [q][a][3] of the 8 trilinear
    functions at the 8 Gauss points; q and a run x fastest."""
    g = _gauss()
    val, grad = np.zeros((8, 8)), np.zeros((8, 8, 3))
    for q in range(8):
        p = [g[q & 1], g[(q >> 1) & 1], g[q >> 2]]
        for a in range(8):
            o = [a & 1, (a >> 1) & 1, a >> 2]
            f = [p[d] if o[d] else 1 - p[d] for d in range(3)]
            val[q, a] = f[0] * f[1] * f[2]
            for d in range(3):
                grad[q, a, d] = (1.0 if o[d] else -1.0) * f[(d + 1) % 3] * f[(d + 2) % 3]
    return val, grad


def _part(t, a, N):
    """Of a nodal field, the values at corner a of every element."""
    x, y, z = a & 1, (a >> 1) & 1, a >> 2
    return t[z:z + N, y:y + N, x:x + N]


class _Stencil:
    """A matrix on the mesh as 27 fields of entries, boundary rows and columns
    of the Dirichlet problem in place."""

    def __init__(self, N, s):
        self.N = N
        self.v = torch.zeros((27, N + 1, N + 1, N + 1, s), dtype=torch.float64, device=DEV)

    def add(self, a, b, ke):
        d = [((b >> t) & 1) - ((a >> t) & 1) + 1 for t in range(3)]
        _part(self.v[d[0] + 3 * d[1] + 9 * d[2]], a, self.N).add_(ke)

    def close(self):
        N, v = self.N, self.v
        inner = torch.zeros((N + 3,) * 3, dtype=torch.float64, device=DEV)
        inner[2:N + 1, 2:N + 1, 2:N + 1] = 1.0
        row = inner[1:N + 2, 1:N + 2, 1:N + 2]
        for t in range(27):
            dx, dy, dz = t % 3, (t // 3) % 3, t // 9
            v[t] *= (row * inner[dz:dz + N + 1, dy:dy + N + 1, dx:dx + N + 1])[..., None]
        v[13] += (1.0 - row)[..., None]
        return self

    def __call__(self, x):
        N = self.N
        p = torch.zeros((N + 3, N + 3, N + 3, x.shape[-1]), dtype=torch.float64, device=DEV)
        p[1:N + 2, 1:N + 2, 1:N + 2] = x
        y = torch.zeros_like(x)
        for t in range(27):
            dx, dy, dz = t % 3, (t // 3) % 3, t // 9
            y.addcmul_(self.v[t], p[dz:dz + N + 1, dy:dy + N + 1, dx:dx + N + 1])
        return y


def _diffusion(N, M, sigma, xi, alpha=0.0, closed=True):
    """D (+ alpha C) of the ensemble, and the load."""
    h, s = 1.0 / N, xi.shape[0]
    val, grad = _shapes()
    A = _Stencil(N, s)
    kap = _Kappa(N, M, sigma, xi)
    for q in range(8):
        k = kap.at(q >> 2, (q >> 1) & 1, q & 1) * (h / 8)
        for a in range(8):
            for b in range(8):
                c = float(grad[q, a] @ grad[q, b])
                if c != 0.0:
                    A.add(a, b, k * c)
    if alpha:
        for a in range(8):
            for b in range(8):
                A.add(a, b, alpha * h * h / 8 * float(sum(val[q, a] * (grad[q, b] @ np.array(VEL)) for q in range(8))))
    load = torch.zeros((N + 1, N + 1, N + 1, s), dtype=torch.float64, device=DEV)
    load[1:N, 1:N, 1:N] = h ** 3
    return (A.close() if closed else A), load


def _dot(a, b):
    return (a * b).sum((0, 1, 2))


def _solve_cg(A, b, tol=1e-14, cap=1500):
    dinv = 1.0 / A.v[13]
    x, r = torch.zeros_like(b), b.clone()
    z = dinv * r
    p, rho, b2 = z.clone(), _dot(r, z), _dot(b, b)
    for it in range(cap):
        q = A(p)
        al = rho / _dot(p, q)
        x.addcmul_(p, al.expand_as(p))
        r.addcmul_(q, (-al).expand_as(q))
        z = dinv * r
        new = _dot(r, z)
        p = z + (new / rho) * p
        rho = new
        if it % 20 == 19 and float((_dot(r, r) / b2).max()) < tol * tol:
            break
    return x


def _solve_bicgstab(A, b, tol, cap=600):
    dinv = 1.0 / A.v[13]
    x, r = torch.zeros_like(b), b.clone()
    r0, p, v = r.clone(), torch.zeros_like(b), torch.zeros_like(b)
    rho = al = om = torch.ones(b.shape[-1], dtype=torch.float64, device=DEV)
    b2 = _dot(b, b)
    for it in range(cap):
        new = _dot(r0, r)
        p = r + (new / rho) * (al / om) * (p - om * v)
        rho = new
        ph = dinv * p
        v = A(ph)
        al = rho / _dot(r0, v)
        sres = r - al * v
        sh = dinv * sres
        t = A(sh)
        om = _dot(t, sres) / _dot(t, t)
        x = x + al * ph + om * sh
        r = sres - om * t
        if it % 10 == 9 and float((_dot(r, r) / b2).max()) < tol * tol:
            break
    return x


def _newton(case, xi):
    N, h, beta = case["N"], 1.0 / case["N"], case["beta"]
    val, _ = _shapes()
    L, load = _diffusion(N, case["M"], case["sigma"], xi, case["alpha"], closed=True)
    u = torch.zeros_like(load)
    inner = (load != 0).to(torch.float64)
    for _ in range(8):
        uq = [sum(val[q, a] * _part(u, a, N) for a in range(8)) for q in range(8)]
        F = L(u) - load
        R = torch.zeros_like(F)
        J = _Stencil(N, xi.shape[0])
        for a in range(8):
            _part(R, a, N).add_(sum(float(val[q, a]) * uq[q] * uq[q] for q in range(8)) * (beta * h ** 3 / 8))
            for b in range(8):
                J.add(a, b, sum(float(val[q, a] * val[q, b]) * uq[q] for q in range(8)) * (beta * h ** 3 / 4))
        J.close()
        J.v[13] -= (1.0 - inner)  # close() made the boundary rows identities; L has them already
        J.v += L.v
        F = (F + R) * inner
        if float((_dot(F, F) / _dot(load, load)).max()) < 1e-26:
            break
        u = u - _solve_bicgstab(J, F, 1e-7)
    return u


def _network(p, x):
    W1, b1 = p[:2560].view(256, 10), p[2560:2816]
    W2, b2 = p[2816:68352].view(256, 256), p[68352:68608]
    W3, b3 = p[68608:76800].view(32, 256), p[76800:76832]
    h = torch.nn.functional.gelu(x @ W1.t() + b1)
    h = torch.nn.functional.gelu(h @ W2.t() + b2)
    return h @ W3.t() + b3


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "spmv"):
        N, s = case["N"], case["s"]
        A, load = _diffusion(N, case["M"], case["sigma"], _xi(seed, s, case["M"]))
        if kind == "spmv":
            x = np.random.default_rng(seed + 1).uniform(-1.0, 1.0, ((N + 1) ** 3, s))
            x = torch.as_tensor(x if case["fp64"] else x.astype(np.float32).astype(np.float64), device=DEV)
            return A(x.view(N + 1, N + 1, N + 1, s)).reshape(-1, s)
        return dict(x=_solve_cg(A, load).reshape(-1, s), rhs=load.reshape(-1, s), iters=None)
    if kind == "newton":
        return dict(u=_newton(case, _xi(seed, case["s"], case["M"])).reshape(-1, case["s"]), iters=None)
    if kind == "batch":
        meshes, s = _meshes(case), case["s"]
        xi = _xi(seed, len(meshes) * s, case["M"]).reshape(len(meshes), s, -1)
        return dict(x=[_solve_cg(*_diffusion(N, case["M"], case["sigma"], xi[i])).reshape(-1, s)
                       for i, N in enumerate(meshes)], iters=[None] * len(meshes))
    if kind == "contrast":
        lo, hi = [], []
        xi = _xi(seed, case["samples"], case["M"])
        for a in range(0, case["samples"], 64):
            kap = _Kappa(case["N"], case["M"], case["sigma"], xi[a:a + 64])
            k = [kap.at(q >> 2, (q >> 1) & 1, q & 1) for q in range(8)]
            lo.append(torch.stack([t.amin((0, 1, 2)) for t in k]).amin(0))
            hi.append(torch.stack([t.amax((0, 1, 2)) for t in k]).amax(0))
        lo, hi = torch.cat(lo), torch.cat(hi)
        return dict(kmin=lo, kmax=hi, order=None)
    if kind == "basis":
        S = _snapshots(case["N"], case["m"], seed)
        lam, V = torch.linalg.eigh((S.t() @ S).cpu())
        lam, V = lam.flip(0)[:32].to(DEV), V.flip(1)[:, :32].to(DEV)
        Phi = (S @ V) / lam.sqrt()
        at = Phi.abs().argmax(0)
        Phi = Phi * torch.sign(Phi.gather(0, at[None, :]))
        C = S.t() @ Phi
        mu = C.mean(0)
        sd = C.std(0, unbiased=False).max().expand(32).contiguous()
        return dict(T=(C - mu) / sd, Phi=Phi, lam=lam, mu=mu, sd=sd)
    if kind == "train":
        count, batch = case["count"], case["batch"]
        xin = _xi(seed, count, ens.MLP_IN)
        x = torch.as_tensor(xin.astype(np.float32).astype(np.float64), device=DEV)
        T = torch.as_tensor(_targets(xin, seed + 1).astype(np.float64), device=DEV)
        p = ens.mlp_init(seed + 2, DEV).double()
        m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
        idx = torch.as_tensor(_order(case, seed).astype(np.int64), device=DEV).view(-1, batch)
        for t in range(case["steps"]):
            p.requires_grad_(True)
            loss = (_network(p, x[idx[t]]) - T[idx[t]]).square().mean()
            gr, = torch.autograd.grad(loss, p)
            p = p.detach()
            m = 0.9 * m + 0.1 * gr
            v = 0.999 * v + 0.001 * gr * gr
            p = p - 1e-3 * (m / (1 - 0.9 ** (t + 1))) / ((v / (1 - 0.999 ** (t + 1))).sqrt() + 1e-8)
            losses.append(loss.detach())
        return dict(params=p, m=m, v=v, loss=torch.stack(losses))
    mu, sd = (torch.as_tensor(v, device=DEV) for v in _scales(seed))
    x = torch.as_tensor(_xi(seed, case["s"], ens.MLP_IN).astype(np.float32).astype(np.float64), device=DEV)
    c = _network(ens.mlp_init(seed + 2, DEV).double(), x)
    return _modes(case["N"], 32, seed) @ (mu + sd * c).t().contiguous()
