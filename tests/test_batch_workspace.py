"""Bytes of a batched solve's workspace, from its layout: the groups'
descriptors, a table entry and two partial ensembles for every tile of rows (a
wavefront's 128 / s rows times `tile`; or of vectors, 1024 chunks of 2 values), two
for each 256 tiles, a control block and four vectors a group, every area
rounded up to 256 bytes.  That much is enough for any solve, as it always was;
at s = 8 the bytes asked for hold four more partial ensembles a tile and for
each 256 tiles.  A solve
with the least workspace adds its partial sums in another order: the same
iterations, or one more or less, to the same solution."""
import ctypes

import numpy as np
import pytest
import torch

from workloads import draw_xi

GROUP, CONTROL, ASSEMBLY = 152, 3376, 80


def _r(b):
    return (b + 255) // 256 * 256


def _rows(meshes, s, tile):
    return [-(-(N + 1) ** 3 // (tile * 128 // s)) for N in meshes]


def _least(meshes, s, tile):
    n = [(N + 1) ** 3 for N in meshes]
    rows = _rows(meshes, s, tile)
    vecs = [-(-(k * s // 2) // 1024) for k in n]
    red, redv = (sum(-(-t // 256) for t in v) for v in (rows, vecs))
    return (_r(GROUP * len(n)) + _r(4 * (sum(rows) + sum(vecs) + red + redv))
            + _r(16 * s * max(sum(rows), sum(vecs))) + _r(16 * s * max(red, redv)) + _r(CONTROL * len(n)) + 256
            + sum(4 * _r(8 * k * s) for k in n))


def _more(meshes, s, tile):
    if s > 8:
        return 0
    rows = _rows(meshes, s, tile)
    return _r(8 * 4 * s * (sum(rows) + sum(-(-t // 256) for t in rows)))


def _assembly(meshes):
    tiles = sum((N // 4 + 1) ** 2 * (N // 2 + 1) for N in meshes)
    return _r(ASSEMBLY * len(meshes)) + _r(4 * tiles)


@pytest.mark.parametrize("s", [8, 16, 32])
@pytest.mark.parametrize("tile", [2, 4, 8])
@pytest.mark.parametrize("meshes", [[2], [16], [31, 64], [32, 48, 64, 96, 48, 32, 64, 48]])
def test_bytes_asked_for_and_refused(s, tile, meshes):
    from paper_1511_03703_amd import batchpool, ens as E
    graphs, groups = [], (E.ens_group * len(meshes))()
    inputs = (E.ens_group_input * len(meshes))()
    stats = (E.ens_cg_stat * s)()
    for i, N in enumerate(meshes):
        graphs.append(E.ens_graph((N + 1) ** 3, (3 * N + 1) ** 3, 256, 256))  # (addresses are not read)
        groups[i] = E.ens_group(ctypes.pointer(graphs[i]), 256, 256, 256, stats)
        inputs[i] = E.ens_group_input(N, 256, 256)
    L, b, opts, prob = E.lib(), ctypes.c_size_t(), E.batch_opts(tile=tile), E.ens_problem(3, 1.0, 1.0, 0.2, 1.0)
    o, p, n = ctypes.byref(opts), ctypes.byref(prob), len(meshes)
    least = _least(meshes, s, tile)
    more = _more(meshes, s, tile)
    assert L.ens_batch_workspace_bytes(groups, n, s, o, ctypes.byref(b)) == E.ENS_OK
    assert b.value == least + more
    assert L.ens_assemble_solve_batch_workspace_bytes(groups, inputs, n, s, p, o, ctypes.byref(b)) == E.ENS_OK
    assert b.value == least + _assembly(meshes) + more
    assert b.value <= sum(batchpool.group_workspace_bound(N, s) for N in meshes)
    # one byte less than the least is refused before any work
    assert L.ens_solve_batch(groups, n, s, o, 256, least - 1, None) == E.ENS_E_NOMEM
    assert L.ens_assemble_solve_batch(groups, inputs, n, s, p, o, 256, least + _assembly(meshes) - 1,
                                      None) == E.ENS_E_NOMEM


@pytest.mark.gpu
@pytest.mark.parametrize("s,tile", [(8, 2), (8, 4), (8, 8), (16, 4)])
def test_solves_with_every_workspace(s, tile):
    from paper_1511_03703_amd import ens as E
    meshes, M, sigma, dev = [12, 5, 31], 4, 0.3, "cuda"
    groups, inputs = [], []
    for i, N in enumerate(meshes):
        g, kl = E.graph_build(N), E.kl_build(N, M)
        xi = torch.as_tensor(draw_xi(40 + i, s, M), device=dev)
        v, _, b = E.assemble(g, kl, xi, M, sigma)
        groups.append([g, v, b, torch.zeros_like(b)])
        inputs.append((N, kl, xi))
    opts = E.batch_opts(rtol=1e-10, tile=tile)
    stats, rc, ws = E.solve_batch(groups, s, opts)
    assert rc == E.ENS_OK
    want = [g[3].clone() for g in groups]
    least = _least(meshes, s, tile)
    for asm in (False, True):
        size = least + (_assembly(meshes) if asm else 0)
        for extra in (0, 255, _more(meshes, s, tile)):
            buf = torch.full((size + extra + 512,), 0x5A, dtype=torch.uint8, device=dev)
            held = buf[:size + extra]
            for g in groups:
                g[3].zero_()
            if asm:
                got, rc, _ = E.assemble_solve_batch(groups, inputs, s, M, sigma, opts, workspace=held,
                                                    strict_workspace=True)
            else:
                got, rc, _ = E.solve_batch(groups, s, opts, workspace=held, strict_workspace=True)
            assert rc == E.ENS_OK
            assert bool((buf[size + extra:] == 0x5A).all())
            for g, x, a, w in zip(groups, want, got, stats):
                same = [p["iters"] == q["iters"] for p, q in zip(a, w)]
                assert all(abs(p["iters"] - q["iters"]) <= 1 for p, q in zip(a, w))
                rel = ((g[3] - x).norm(dim=0) / x.norm(dim=0)).cpu().numpy()
                assert (rel <= np.where(same, 1e-10, 1e-8)).all()
    with pytest.raises(E.EnsError) as ex:
        E.solve_batch(groups, s, opts, workspace=ws[:least - 1], strict_workspace=True)
    assert ex.value.status == E.ENS_E_NOMEM


@pytest.mark.gpu
def test_autotuner_with_the_least_workspace():
    from paper_1511_03703_amd import ens as E
    meshes, M = (ctypes.c_int32 * 2)(6, 9), 3
    sc, tc = (ctypes.c_int32 * 1)(8), (ctypes.c_int32 * 1)(4)
    prob, opts = E.ens_problem(M, 1.0, 1.0, 0.2, 1.0), E.batch_opts()
    xi = np.ascontiguousarray(np.stack([draw_xi(60 + i, 32, M) for i in range(2)]))
    need, s, t = ctypes.c_size_t(), ctypes.c_int32(), ctypes.c_int32()
    L = E.lib()
    shape = (ctypes.addressof(meshes), 2, ctypes.byref(prob))
    cand = (ctypes.addressof(sc), 1, ctypes.addressof(tc), 1, ctypes.byref(opts))
    assert L.ens_batch_autotune_workspace_bytes(*shape, *cand, ctypes.byref(need)) == E.ENS_OK
    more = _more([6] * 4 + [9] * 4, 8, 4)
    ws = torch.empty(need.value, dtype=torch.uint8, device="cuda")
    score = (ctypes.c_double * 1)()
    for size, ok in ((need.value, True), (need.value - more, True), (need.value - more - 1, False)):
        score[0] = -1.0
        rc = L.ens_batch_autotune(*shape, xi.ctypes.data, *cand, None, ctypes.byref(s), ctypes.byref(t),
                                  ctypes.addressof(score), ws.data_ptr(), size, E._stream())
        assert (rc == E.ENS_OK) == ok, size
        assert (score[0] > 0.0) == ok
