"""The network's rows kernel at its edges: one row per workgroup (up to one per CU),
four with every remainder, the switch to layer-wise products in the forward pass, and
parameters and features at addresses of four bytes only, against the FP64 oracle
(1e-4 relative: sums of 258 products in FP32 err by at most 258 2^-24 = 1.6e-5)."""
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


def _odd(a):
    """Contiguous CUDA copy of a whose address is 4 modulo 16."""
    t = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")[1:].view(a.shape)
    return t.copy_(torch.from_numpy(np.ascontiguousarray(a)))


@pytest.mark.parametrize("B", [1, 2, 256, 257, 258, 259, 260, 1027, 16384, 16385])
def test_rows_kernel_edges(P, B):
    rng = np.random.default_rng(B)
    X = rng.uniform(-1, 1, (B, OM.D_IN)).astype(np.float32)
    T = rng.standard_normal((B, OM.D_OUT)).astype(np.float32)
    theta = OM.init_params(B).astype(np.float32)
    p, x, t = _odd(theta), _odd(X), _odd(T)
    assert p.data_ptr() % 16 == 4 and x.data_ptr() % 16 == 4
    y = P.chebfd_mlp_forward(p, x).cpu().numpy()
    ref, _ = OM.forward(theta.astype(np.float64), X.astype(np.float64))
    assert np.max(np.abs(y - ref)) <= 1e-4 * max(1.0, np.max(np.abs(ref)))
    loss, g = P.chebfd_mlp_grad(p, x, t)
    rl, rg = OM.gradient(theta.astype(np.float64), X.astype(np.float64), T.astype(np.float64))
    assert abs(loss.item() - rl) <= 1e-4 * abs(rl)
    g, at = g.cpu().numpy(), 0
    for s in OM.SHAPES:
        k = int(np.prod(s))
        assert np.max(np.abs(g[at:at + k] - rg[at:at + k])) <= 1e-4 * max(np.max(np.abs(rg[at:at + k])), 1e-30), s
        at += k
