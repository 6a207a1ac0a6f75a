"""The TGV kernel's tiles against the FP64 oracle: each number of lanes of a row and the sizes beside it, rows cut into
several tiles along z, the last full and the first partial tile along y and x, and volumes of one voxel's width.
Tolerance: differences of FP32 inputs, a hardware square root and reciprocal of 1 ulp, and sums of at most nine terms,
about 5 roundings of 6e-8 each; 1e-6 leaves a factor of three."""
import numpy as np
import pytest

from gpu_helpers import announce, rel_l2
from oracle import oracle as O

pytestmark = pytest.mark.gpu
A0, A1, EPS, TOL = 0.6, 1.1, 1e-2, 1e-6


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 3), (3, 1, 1), (2, 46, 64), (3, 47, 63), (5, 23, 65), (4, 22, 128),
                                   (9, 11, 129), (300, 10, 7), (2, 3, 256), (3, 12, 257), (2, 5, 497), (6, 21, 252)])
def test_tgv_tiles(shape):
    import torch
    from paper_2604_09643_amd import _lib as L
    announce("tgv tiles %s" % (shape,))
    rng = np.random.default_rng(sum(shape))
    u = rng.normal(size=shape).astype(np.float32)
    w = (0.3 * rng.normal(size=(3,) + shape)).astype(np.float32)
    # one voxel into a larger allocation: nothing but FP32 alignment is promised
    ut = torch.zeros(u.size + 1, device="cuda:0")[1:].view(shape).copy_(torch.tensor(u))
    wt = torch.zeros(w.size + 1, device="cuda:0")[1:].view(w.shape).copy_(torch.tensor(w))
    guard = torch.full((2 * u.size + w.size * 2 + 64,), 7.0, device="cuda:0")
    gu = guard[17:17 + u.size].view(shape)
    gw = guard[33 + u.size:33 + u.size + w.size].view(w.shape)
    val = L.tgv_loss_and_grad(ut, wt, A0, A1, EPS, scale=0.5, grad_u=gu, grad_w=gw)
    ref = 0.5 * O.tgv_value(u, w, A0, A1, EPS)
    gu_ref, gw_ref = O.tgv_grad(u, w, A0, A1, EPS)
    assert abs(val - ref) <= TOL * abs(ref)
    assert np.abs(gu.cpu().numpy() - 0.5 * gu_ref).max() <= TOL * max(1.0, np.abs(gu_ref).max())
    assert rel_l2(gw.cpu().numpy(), 0.5 * gw_ref) <= TOL
    L.tgv_loss_and_grad(ut, wt, A0, A1, EPS, scale=0.25, want_loss=False, grad_w=gw, accumulate=True)
    assert rel_l2(gw.cpu().numpy(), 0.75 * gw_ref) <= TOL
    host = guard.cpu().numpy()
    host[17:17 + u.size] = 7.0
    host[33 + u.size:33 + u.size + w.size] = 7.0
    assert (host == 7.0).all()
    assert L.tgv_loss_and_grad(ut, wt, A0, A1, EPS, scale=0.5) == val


def test_tgv_infinite_input_stays_local():
    """An infinite u beside the boundary reaches only the voxels whose differences hold it."""
    import torch
    from paper_2604_09643_amd import _lib as L
    announce("tgv infinite input")
    u = torch.zeros((6, 30, 70), device="cuda:0")
    u[0, 0, 0] = float("inf")
    w = torch.ones((3, 6, 30, 70), device="cuda:0")
    gu, gw = torch.empty_like(u), torch.empty_like(w)
    L.tgv_loss_and_grad(u, w, A0, A1, EPS, want_loss=False, grad_u=gu, grad_w=gw)
    bad = (~torch.isfinite(gw)).any(0).nonzero().tolist()
    assert bad == [[0, 0, 0]]
    assert sorted((~torch.isfinite(gu)).nonzero().tolist()) == [[0, 0, 0], [0, 0, 1], [0, 1, 0], [1, 0, 0]]
