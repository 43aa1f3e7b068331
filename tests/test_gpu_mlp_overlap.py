"""Network calls whose buffers lie inside one another: the outputs of the forward pass
inside the features or the first layers' parameters (both are read before the last
layer writes), against the FP64 oracle (1e-4 relative: sums of 258 products in FP32 err
by at most 258 2^-24 = 1.6e-5); the loss inside the gradient or the targets (the gradient
is whole, the same bits as with a loss of its own)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle.mlp as OM

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1803_02156_amd as P
    P.load()
    return P


def _ptr(t, floats=0):
    return ctypes.c_void_p(t.data_ptr() + 4 * floats)


def _work(P, batch):
    sz = ctypes.c_size_t()
    P.check(P.load().chebfd_mlp_query(batch, None, ctypes.byref(sz)))
    return P.device_buffer(sz.value), sz.value


def _inputs(B):
    rng = np.random.default_rng(B)
    X = rng.uniform(-1, 1, (B, OM.D_IN)).astype(np.float32)
    T = rng.standard_normal((B, OM.D_OUT)).astype(np.float32)
    return OM.init_params(B).astype(np.float32), X, T


@pytest.mark.parametrize("B", [1, 7, 300, 1027, 16384])
@pytest.mark.parametrize("where", ["start", "middle", "end", "params"])
def test_forward_outputs_inside_inputs(P, B, where):
    theta, X, _ = _inputs(B)
    if where == "params" and OM.D_OUT * B > 128 * 258:
        pytest.skip("the outputs are longer than the first layer's weights")
    ref, _ = OM.forward(theta.astype(np.float64), X.astype(np.float64))
    p, x = torch.from_numpy(theta.copy()).cuda(), torch.from_numpy(X.copy()).cuda()
    at = {"start": 0, "middle": (X.size - ref.size) // 2, "end": X.size - ref.size, "params": 0}[where]
    into = p if where == "params" else x.view(-1)
    work, nbytes = _work(P, B)
    for _ in range(3):
        p.copy_(torch.from_numpy(theta))
        x.copy_(torch.from_numpy(X))
        P.check(P.load().chebfd_mlp_forward(_ptr(p), B, _ptr(x), _ptr(into, at), _ptr(work), nbytes, P.chebfd._stream()))
        y = into[at:at + ref.size].view(B, OM.D_OUT).cpu().numpy()
        assert np.max(np.abs(y - ref)) <= 1e-4 * max(1.0, np.max(np.abs(ref)))


@pytest.mark.parametrize("B", [1, 125, 1027])
@pytest.mark.parametrize("at", [0, 33023, 33024, 49920, 49921])
def test_loss_inside_gradient(P, B, at):
    theta, X, T = _inputs(B)
    p, x, t = (torch.from_numpy(v).cuda() for v in (theta, X, T))
    _, ref = P.chebfd_mlp_grad(p, x, t)
    work, nbytes = _work(P, B)
    for _ in range(3):
        g = torch.full_like(ref, float("nan"))
        P.check(P.load().chebfd_mlp_grad(_ptr(p), B, _ptr(x), _ptr(t), _ptr(g, at), _ptr(g), _ptr(work), nbytes,
                                         P.chebfd._stream()))
        assert torch.equal(g, ref)


@pytest.mark.parametrize("B", [1, 125, 1027])
def test_loss_inside_targets(P, B):
    theta, X, T = _inputs(B)
    p, x, t = (torch.from_numpy(v).cuda() for v in (theta, X, T))
    loss, ref = P.chebfd_mlp_grad(p, x, t)
    work, nbytes = _work(P, B)
    g = torch.full_like(ref, float("nan"))
    P.check(P.load().chebfd_mlp_grad(_ptr(p), B, _ptr(x), _ptr(t), _ptr(t, 2 * B - 1), _ptr(g), _ptr(work), nbytes,
                                     P.chebfd._stream()))
    assert torch.equal(g, ref) and t.view(-1)[2 * B - 1] == loss[0]
