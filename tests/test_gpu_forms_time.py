"""Which form a call takes where one is much slower than the other: coarse spacings, small regions with edge terms.
Times are medians of several runs and compared with another call's of the same form, with room for a box's mood."""
import time

import pytest

from gpu_helpers import announce
from paper_2604_09643_amd import workloads as W

pytestmark = pytest.mark.gpu


def median_us(f, runs=9, each=5):
    import torch
    f()
    t = []
    for _ in range(runs):
        torch.cuda.synchronize()
        a = time.perf_counter()
        for _ in range(each):
            f()
        torch.cuda.synchronize()
        t.append((time.perf_counter() - a) / each)
    return sorted(t)[runs // 2] * 1e6


def setup(h, sigma, n=40, kernel=0, trunc=6.0, M=64, F=4, K=2048):
    import torch
    from paper_2604_09643_amd import _lib as L
    dev = "cuda:0"
    gen = torch.Generator(device=dev).manual_seed(1)
    g = L.Grid(n, n, n, (-0.5 * (n - 1) * h, -0.5 * (n - 1) * h, 6e-3), h)
    s = L.Sampling(1540.0, 40e6, K, sigma, trunc, kernel, 2.0)
    p = torch.randn((n, n, n), generator=gen, device=dev)
    elem = torch.tensor(W.linear_array(M, 3e-4), dtype=torch.float64, device=dev)
    poses = torch.zeros((F, 12), dtype=torch.float64, device=dev)
    poses[:, 0] = poses[:, 4] = poses[:, 8] = 1.0
    poses[:, 11] = -1e-4 * torch.arange(F, device=dev)
    r = torch.randn((F, M, K), generator=gen, device=dev)
    return L, g, s, p, elem, poses, r


@pytest.mark.parametrize("sigma,h,n,F", [(1e-4, 5e-4, 40, 4), (6e-5, 4.2e-4, 40, 4), (8e-5, 4.2e-4, 96, 1)])
def test_coarse_forward_takes_the_row_form(sigma, h, n, F):
    """The negative-correlation loss always runs the row form, and its statistics; the moment form took 2.9 to 3.7 times that."""
    import torch
    L, g, s, p, elem, poses, r = setup(h, sigma, n, F=F)
    announce("coarse forward sigma %g h %g" % (sigma, h))
    out = torch.empty_like(r)
    fwd = median_us(lambda: L.radiate_forward(g, p, elem, poses, s, s=out))
    nc = median_us(lambda: L.nc_loss_and_grad(g, p, elem, poses, s, r))
    assert fwd <= 1.3 * nc, (fwd, nc)


@pytest.mark.parametrize("sigma,h", [(1e-4, 4.2e-4), (1e-4, 6e-4)])
def test_coarse_volume_adjoint(sigma, h):
    """dL/dp0 alone is less work than with the element gradients; on the row form's small regions it took twice as long."""
    import torch
    L, g, s, p, elem, poses, r = setup(h, sigma)
    announce("coarse adjoint sigma %g h %g" % (sigma, h))
    gp, ge = torch.empty_like(p), torch.empty((4, 64, 3), dtype=torch.float64, device="cuda:0")
    one = median_us(lambda: L.radiate_adjoint(g, None, elem, poses, s, r, grad_p0=gp))
    both = median_us(lambda: L.radiate_adjoint(g, p, elem, poses, s, r, grad_p0=gp, grad_elem=ge))
    assert one <= 1.2 * both, (one, both)


def test_small_regions_occupy_all_wavefronts():
    """The exponential's adjoint has fewer terms than the power law's; 4 of 16 wavefronts at work made it 1.2 times as long."""
    import torch
    announce("edge-term adjoints")
    t = {}
    for kernel, trunc in ((1, 12.0), (2, 10.0)):
        L, g, s, p, elem, poses, r = setup(1e-4, 8e-5, kernel=kernel, trunc=trunc)
        gp = torch.empty_like(p)
        t[kernel] = median_us(lambda: L.radiate_adjoint(g, None, elem, poses, s, r, grad_p0=gp))
    assert t[1] <= 1.1 * t[2], t
