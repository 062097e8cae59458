"""Solves on several threads of one process at once, each with its own stream,
graph and workspace: every one gives bitwise what it gives alone (a poll
decides when a solve ends, when it moves to a compacted ensemble and when it
polls again, never what an iteration computes).  Batches and the concurrent
one-sample baseline, which work on streams of the device's context, take turns
there."""
import threading

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


def _job(E, k):
    """A solve as a closure of its stream; short and long ones, of every loop
    that polls through the library's pinned words."""
    N, s, M = ((8, 4, 3), (24, 16, 5), (16, 8, 10), (20, 8, 4))[k]
    g, kl = E.graph_build(N), E.kl_build(N, M)
    xi = torch.as_tensor(draw_xi(500 + k, s, M), device=DEV)
    v, v32, b = E.assemble(g, kl, xi, M, 0.3, want32=True)
    mg = E.Multigrid(N, M, s).setup(g, v, xi, 0.3) if k == 2 else None
    opts = E.cg_opts(rtol=1e-10, check_every=1 if k == 0 else 3, compact=k == 1, mixed=k == 3)
    nb = E.cg_workspace_bytes(g, s, opts)
    ws = torch.empty(nb, dtype=torch.uint8, device=DEV)

    def solve(stream):
        x = torch.zeros_like(b)
        stream.wait_stream(torch.cuda.current_stream())
        if mg is not None:
            out = E.cg_mg(g, v, b, mg, x=x, opts=opts, workspace=ws, stream=stream)
        else:
            out = E.cg(g, v, b, x=x, values32=v32 if opts.mixed else None, opts=opts, workspace=ws, stream=stream)
        stream.synchronize()
        return out

    return solve


def test_solves_side_by_side(E):
    jobs = [_job(E, k) for k in range(4)]
    streams = [torch.cuda.Stream() for _ in jobs]
    torch.cuda.synchronize()
    alone = [job(st) for job, st in zip(jobs, streams)]
    wrong = []

    def work(k):
        try:
            torch.cuda.set_device(0)
            for n in range(12):
                x, stats, rc = jobs[k](streams[k])
                if rc != alone[k][2] or stats != alone[k][1] or not torch.equal(x, alone[k][0]):
                    wrong.append((k, n, rc, [t["iters"] for t in stats]))
        except Exception as e:  # noqa: BLE001
            wrong.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(rc == E.ENS_OK for _, _, rc in alone)
    assert not wrong, wrong[:5]


def _shared_job(E, k):
    """A batch (captured or launched) or a concurrent baseline as a closure of its stream."""
    if k == 3:
        N, s, M = 10, 6, 3
        g, kl = E.graph_build(N), E.kl_build(N, M)
        v, _, b = E.assemble(g, kl, torch.as_tensor(draw_xi(610, 8, M), device=DEV), M, 0.3)
        vs, bs = v.t()[:s].contiguous(), b.t()[:s].contiguous()

        def solve(stream):
            x = torch.zeros_like(bs)
            stream.wait_stream(torch.cuda.current_stream())
            out = E.scalar_cg_concurrent(g, vs, bs, x_sm=x, opts=E.cg_opts(rtol=1e-10), streams=4, stream=stream)
            stream.synchronize()
            return [out[0]], out[1], out[2]

        return solve
    meshes, s, M = ([6, 9], [16, 5, 7], [12])[k], (8, 16, 32)[k], 4
    groups, inputs = [], []
    for i, N in enumerate(meshes):
        g, kl = E.graph_build(N), E.kl_build(N, M)
        xi = torch.as_tensor(draw_xi(600 + 10 * k + i, s, M), device=DEV)
        v, _, b = E.assemble(g, kl, xi, M, 0.3)
        groups.append([g, v, b, torch.zeros_like(b)])
        inputs.append((N, kl, xi))
    opts = E.batch_opts(rtol=1e-10, check_every=(2, 5, 3)[k], use_graph=k != 1)

    def solve(stream):
        stream.wait_stream(torch.cuda.current_stream())
        stats, rc, _ = E.assemble_solve_batch(groups, inputs, s, M, 0.3, opts, stream=stream)
        stream.synchronize()
        return [q[3].clone() for q in groups], stats, rc

    return solve


def test_batches_and_the_concurrent_baseline_side_by_side(E):
    jobs = [_shared_job(E, k) for k in range(4)]
    streams = [torch.cuda.Stream() for _ in jobs]
    torch.cuda.synchronize()
    alone = [job(st) for job, st in zip(jobs, streams)]
    torch.cuda.synchronize()
    wrong = []

    def work(k):
        try:
            torch.cuda.set_device(0)
            for n in range(8):
                xs, stats, rc = jobs[k](streams[k])
                torch.cuda.current_stream().synchronize()
                if rc != alone[k][2] or stats != alone[k][1] or not all(map(torch.equal, xs, alone[k][0])):
                    wrong.append((k, n, rc))
        except Exception as e:  # noqa: BLE001
            wrong.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(rc == E.ENS_OK for _, _, rc in alone)
    assert not wrong, wrong[:5]
