"""Network outputs written where the inputs, the targets or the parameters lie:
bitwise what separate buffers give (every workgroup's inputs are read before
outputs replace them)."""
import ctypes

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


def _inputs(E, B):
    g = np.random.default_rng(B)
    xi = torch.as_tensor(g.uniform(-1, 1, (B, E.MLP_IN)).astype(np.float32), device=DEV)
    t = torch.as_tensor(g.standard_normal((B, E.MLP_OUT)).astype(np.float32), device=DEV)
    return E.mlp_init(3, DEV), xi, t


def _ptr(t, floats=0):
    return ctypes.c_void_p(t.data_ptr() + 4 * floats)


@pytest.mark.parametrize("B", [32, 2048, 8192])
def test_outputs_over_inputs(E, B):
    params, xi, t = _inputs(E, B)
    L, st, ws = E.lib(), E._stream(), E._mlp_ws(B, DEV)
    want, grad, loss = E.mlp_grad(params, xi, t)
    assert torch.equal(E.mlp_forward(params, xi), want)
    n_in, n_out = B * E.MLP_IN, B * E.MLP_OUT
    for shift in (0, n_out - n_in, n_out - 1):  # the inputs' start in the outputs
        buf = torch.zeros(2 * n_out, device=DEV)
        buf[shift:shift + n_in] = xi.ravel()
        assert L.ens_mlp_forward(_ptr(params), B, _ptr(buf, shift), _ptr(buf), _ptr(ws), ws.numel(), st) == E.ENS_OK
        assert torch.equal(buf[:n_out].view(B, -1), want)
        buf.zero_()
        buf[shift:shift + n_in] = xi.ravel()
        g2, l2 = torch.empty_like(grad), torch.empty_like(loss)
        assert L.ens_mlp_grad(_ptr(params), B, _ptr(buf, shift), _ptr(t), _ptr(buf), _ptr(g2), _ptr(l2), _ptr(ws),
                              ws.numel(), st) == E.ENS_OK
        assert torch.equal(buf[:n_out].view(B, -1), want) and torch.equal(g2, grad) and torch.equal(l2, loss)


@pytest.mark.parametrize("B", [32, 2048])
def test_outputs_over_targets_and_parameters(E, B):
    params, xi, t = _inputs(E, B)
    L, st, ws = E.lib(), E._stream(), E._mlp_ws(B, DEV)
    want, grad, loss = E.mlp_grad(params, xi, t)
    n_out = B * E.MLP_OUT
    for shift in (0, 32, n_out // 2):  # the targets' start in the outputs
        buf = torch.zeros(2 * n_out, device=DEV)
        buf[shift:shift + n_out] = t.ravel()
        g2, l2 = torch.empty_like(grad), torch.empty_like(loss)
        assert L.ens_mlp_grad(_ptr(params), B, _ptr(xi), _ptr(buf, shift), _ptr(buf), _ptr(g2), _ptr(l2), _ptr(ws),
                              ws.numel(), st) == E.ENS_OK
        assert torch.equal(buf[:n_out].view(B, -1), want) and torch.equal(g2, grad) and torch.equal(l2, loss)
    buf = torch.zeros(max(n_out, params.numel()), device=DEV)
    buf[:params.numel()] = params
    assert L.ens_mlp_forward(_ptr(buf), B, _ptr(xi), _ptr(buf), _ptr(ws), ws.numel(), st) == E.ENS_OK
    assert torch.equal(buf[:n_out].view(B, -1), want)
