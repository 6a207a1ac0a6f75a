"""Scratch: what a forward-only call takes, and adjoints without room for their moment table."""
import numpy as np
import pytest

from gpu_helpers import announce, rel_l2
from paper_2604_09643_amd import workloads as W

pytestmark = pytest.mark.gpu


def setup(M, F, K, kernel=2, trunc=10.0, sigma=8e-5, shape=(16, 12, 20)):
    import torch
    from paper_2604_09643_amd import _lib as L
    rng = np.random.default_rng(4)
    g, s = L.Grid(*shape, (0.0, 0.0, 5e-3), 1e-4), L.Sampling(1540.0, 40e6, K, sigma, trunc, kernel, 2.0)
    dev = "cuda:0"
    p = torch.tensor(rng.uniform(-0.5, 1.0, shape).astype(np.float32), device=dev)
    elem = torch.tensor(W.linear_array(M, 1e-5), dtype=torch.float64, device=dev)
    poses = torch.zeros((F, 12), dtype=torch.float64, device=dev)
    poses[:, 0] = poses[:, 4] = poses[:, 8] = 1.0
    poses[:, 11] = -1e-5 * torch.arange(F, device=dev)
    return L, g, s, p, elem, poses


@pytest.mark.parametrize("kernel,trunc,sigma", [(2, 10.0, 8e-5), (1, 12.0, 8e-5), (0, 6.0, 6.4e-5)])
def test_forward_takes_no_table(kernel, trunc, sigma):
    """64 MB of signals: their FP64 sums, FP32 copy and tables of positions, but not 800 MB of moment table."""
    import torch
    L, g, s, p, elem, poses = setup(128, 64, 2048, kernel, trunc, sigma)
    announce("scratch of a forward, kernel %d" % kernel)
    out = torch.empty((64, 128, 2048), device="cuda:0")
    ctx = L.Context(0)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    L.radiate_forward(g, p, elem, poses, s, s=out, ctx=ctx)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 300 << 20
    ctx.close()


@pytest.mark.parametrize("kernel,trunc,sigma", [(2, 10.0, 8e-5), (0, 6.0, 8e-5)])
def test_adjoint_without_room_for_its_table(kernel, trunc, sigma):
    """Under capture nothing can be allocated: with scratch for the row form alone the row form runs."""
    import torch
    L, g, s, p, elem, poses = setup(64, 8, 2048, kernel, trunc, sigma)
    announce("adjoint without table, kernel %d" % kernel)
    r = torch.tensor(np.random.default_rng(5).normal(size=(8, 64, 2048)).astype(np.float32), device="cuda:0")
    want, we = torch.empty_like(p), torch.empty((8, 64, 3), dtype=torch.float64, device="cuda:0")
    L.radiate_adjoint(g, p, elem, poses, s, r, grad_p0=want, grad_elem=we)
    ctx = L.Context(0)
    assert ctx.lib.ra_reserve(ctx.ptr, 16 << 20) == L.RA_OK      # signals 4 MB, partials 0.3 MB; tables 33 to 50 MB
    got, ge = torch.empty_like(p), torch.empty_like(we)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        L.radiate_adjoint(g, p, elem, poses, s, r, grad_p0=want.clone(), grad_elem=we.clone())   # kernels loaded
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            L.radiate_adjoint(g, p, elem, poses, s, r, grad_p0=got, grad_elem=ge, ctx=ctx)
    for _ in range(3):
        got.zero_()
        ge.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert rel_l2(got.cpu().numpy(), want.cpu().numpy()) <= 1e-5
        assert rel_l2(ge.cpu().numpy(), we.cpu().numpy()) <= 2e-5
    ctx.close()
