"""Adjoints of narrow Gaussians with windows below 6 sigma against the windowed sum of the FP64 oracle: what lies
between the window's edge and half a sample past its last whole sample is left out (1e-2 to 1e-3 of the peak here)."""
import numpy as np
import pytest

from gpu_helpers import announce, gpu_desc, oracle_desc, rel_l2, to_gpu
from oracle import oracle as O
from paper_2604_09643_amd import workloads as W

pytestmark = pytest.mark.gpu

# rounding of the row forms 3e-6; a term within rounding of the edge (one pair in 1e6) may fall either way, which moves
# a sum over thousands of pairs by less than 1e-5
TOL = 2e-5


@pytest.mark.parametrize("sigma,trunc", [(6e-5, 3.5), (6e-5, 4.0), (5e-5, 4.0), (4e-5, 4.0)])
def test_adjoints_keep_the_window(sigma, trunc):
    import torch
    from paper_2604_09643_amd import _lib as L
    announce("short window sigma %g trunc %g" % (sigma, trunc))
    w = W.small(shape=(21, 17, 19), h=1e-4, M=20, F=1, K=500, sigma=sigma)
    w.trunc = trunc
    (g, s), (p, elem, poses) = gpu_desc(w), to_gpu(w)
    r = w.extra["r"].astype(np.float32)
    rt = torch.tensor(r, device="cuda:0")
    gv, gp, ge = torch.empty_like(p), torch.empty_like(p), torch.empty((1, 20, 3), dtype=torch.float64, device="cuda:0")
    L.radiate_adjoint(g, None, elem, poses, s, rt, grad_p0=gv)
    L.radiate_adjoint(g, p, elem, poses, s, rt, grad_p0=gp, grad_elem=ge)
    og, os_ = oracle_desc(w)
    rd = r.astype(np.float64)
    rp = O.grid_adjoint_p0(og, w.poses, w.elem, os_, rd)
    re = O.grid_adjoint_elem(og, w.p0.astype(np.float32).astype(np.float64), w.poses, w.elem, os_, rd)
    assert rel_l2(gv.cpu().numpy(), rp) <= TOL and rel_l2(gp.cpu().numpy(), rp) <= TOL
    assert rel_l2(ge.cpu().numpy(), re) <= TOL


def test_batched_volume_update_keeps_the_window():
    import torch
    from paper_2604_09643_amd import _lib as L
    from paper_2604_09643_amd.serve import VOLUME, GpuExecutor, Request, Scheduler
    announce("short window batch")
    n, h, M, K, sigma, trunc = 20, 1.1e-4, 16, 400, 6e-5, 4.0           # on 8x8x8 regions
    origin = (-0.5 * (n - 1) * h, -0.5 * (n - 1) * h, 3e-3)
    rng = np.random.default_rng(7)
    vol = rng.uniform(-0.3, 1.0, (n, n, n)).astype(np.float32)
    y = rng.normal(0, 1.0, (M, K)).astype(np.float32)
    ex = GpuExecutor(torch.tensor(vol, device="cuda:0"), L.Grid(n, n, n, origin, h),
                     L.Sampling(1540.0, 40e6, K, sigma, trunc), slots=2, arena_bytes=1 << 26, graph=False, apply_updates=False)
    sch = Scheduler(ex, 2, 1 << 40)
    sch.submit(Request(0, VOLUME, (0, 0, 0, n, n, n), W.linear_array(M, 3e-4), np.zeros(6), y, 2))
    sch.tick()
    st = list(ex.state.values())[0]
    og, os_ = O.Grid(n, n, n, np.array(origin), h), O.Sampling(1540.0, 40e6, K, sigma, trunc)
    poses = np.array([[1.0, 0, 0, 0, 1.0, 0, 0, 0, 1.0, 0, 0, 0]])
    elem = W.linear_array(M, 3e-4)
    # dL/ds as the step left it: the batch's forward takes its rows whole, and more of them where it pairs voxels
    o = st["offs"]["s"]
    r = ex.buf[o:o + 4 * M * K].view(torch.float32).cpu().numpy().astype(np.float64).reshape(1, M, K)
    ref = O.grid_adjoint_p0(og, poses, elem, os_, r)
    assert rel_l2(st["grad"].cpu().numpy(), ref) <= TOL
