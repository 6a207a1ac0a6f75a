"""<A p, r> = <p, A^T r> for the profiles that do not vanish at their window's edge, where every pair of a voxel and an
element lies within rounding of that edge: both directions have to put its outermost sample in or out alike."""
import numpy as np
import pytest

from gpu_helpers import announce

pytestmark = pytest.mark.gpu

# rounding of a signal 1e-6; an edge decided differently for half of the pairs moves the product by 1e-4 (exponential)
# to 1e-3 (power law) of |A p| here
TOL = 1e-5


@pytest.mark.parametrize("kernel,trunc", [(1, 12.0), (2, 10.0)])
@pytest.mark.parametrize("shape", [(1, 1, 160), (2, 3, 77), (9, 9, 77), (17, 4, 130), (6, 20, 160)])
def test_edges_fall_alike(kernel, trunc, shape):
    import torch
    from paper_2604_09643_amd import _lib as L
    announce("edge transpose kernel %d %s" % (kernel, shape))
    delta, sigma, M, K = 1540.0 / 40e6, 8e-5, 64, 900
    h = 2 * delta                          # all on one axis: a voxel's distance is the window's half-width and whole samples
    elem = np.array([[0.0, 0.0, -(trunc * sigma + (40 + m) * delta)] for m in range(M)])
    rng = np.random.default_rng(5)
    dev = "cuda:0"
    p = torch.tensor(rng.normal(size=shape).astype(np.float32), device=dev)
    r = torch.tensor(rng.normal(size=(1, M, K)).astype(np.float32), device=dev)
    g, s = L.Grid(*shape, (0.0, 0.0, 0.0), h), L.Sampling(1540.0, 40e6, K, sigma, trunc, kernel, 2.0)
    et = torch.tensor(elem, device=dev)
    poses = torch.tensor([[1.0, 0, 0, 0, 1.0, 0, 0, 0, 1.0, 0, 0, 0]], dtype=torch.float64, device=dev)
    sig = L.radiate_forward(g, p, et, poses, s).double()
    one, both = torch.empty_like(p), torch.empty_like(p)
    L.radiate_adjoint(g, None, et, poses, s, r, grad_p0=one)
    L.radiate_adjoint(g, p, et, poses, s, r, grad_p0=both, grad_elem=torch.empty((1, M, 3), dtype=torch.float64, device=dev))
    lhs = float((sig * r.double()).sum())
    for grad in (one, both):
        assert abs(lhs - float((p.double() * grad.double()).sum())) <= TOL * float(sig.norm())
