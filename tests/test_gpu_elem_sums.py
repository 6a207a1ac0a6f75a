"""Element gradients whose large terms cancel: four voxels' terms add in single precision, those sums in double."""
import numpy as np
import pytest

from gpu_helpers import announce, rel_l2
from oracle import oracle as O

pytestmark = pytest.mark.gpu

# the terms' own rounding (1e-6) and the double sums' of the large ones, 1e-16 of 1e9 times what is left
TOL = 1e-5


@pytest.mark.parametrize("kernel,trunc", [(0, 6.0), (2, 10.0)])
def test_faint_terms_survive_bright_ones(kernel, trunc):
    """Two mirrored columns of voxels with an element on the plane between them: voxels of +-1e9 cancel along y and z."""
    import torch
    from paper_2604_09643_amd import _lib as L
    announce("element sums kernel %d" % kernel)
    h, sigma, K, M = 1e-4, 8e-5, 400, 6
    rng = np.random.default_rng(2)
    p0 = np.zeros((2, 1, 8), dtype=np.float32)
    p0[0, 0, 1], p0[1, 0, 1] = 1e9, -1e9
    p0[:, 0, 4:] = rng.uniform(0.5, 1.0, (2, 4))
    elem = np.stack([np.zeros(M), np.linspace(-1e-3, 1.5e-3, M), np.full(M, -2e-3)], 1)
    r = rng.normal(size=(1, M, K)).astype(np.float32)
    poses = np.array([[1.0, 0, 0, 0, 1.0, 0, 0, 0, 1.0, 0, 0, 0]])
    origin = (-0.5 * h, 0.0, 0.0)
    g, s = L.Grid(2, 1, 8, origin, h), L.Sampling(1540.0, 40e6, K, sigma, trunc, kernel, 2.0)
    pt, et, qt, rt = (torch.tensor(a, device="cuda:0") for a in (p0, elem, poses, r))
    ge = torch.empty((1, M, 3), dtype=torch.float64, device="cuda:0")
    L.radiate_adjoint(g, pt, et, qt, s, rt, grad_elem=ge)
    p0[:, 0, 1] = 0.0                      # the oracle without the cancelling pair
    ref = O.grid_adjoint_elem(O.Grid(2, 1, 8, np.array(origin), h), p0.astype(np.float64), poses, elem,
                              O.Sampling(1540.0, 40e6, K, sigma, trunc, kernel, 2.0), r.astype(np.float64))
    assert rel_l2(ge.cpu().numpy()[..., 1:], ref[..., 1:]) <= TOL
