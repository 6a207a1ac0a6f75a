"""The batched step on regions of 16 voxels along z (fine spacings: their adjoints run as two of 8) and on regions of few
voxels (coarse: row-form forward, series adjoints) against the single calls, with boxes that leave remainders."""
import time

import numpy as np
import pytest

from gpu_helpers import announce, rel_l2
from paper_2604_09643_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sigma,h,rz,moment", [(1e-4, 5e-5, 16, 1), (1.2e-4, 3e-5, 16, 1), (1e-4, 4e-4, 4, 2)])
def test_batch_equals_single_calls(sigma, h, rz, moment):
    import torch
    from paper_2604_09643_amd import _lib as L
    from paper_2604_09643_amd.serve import POSE, VOLUME, GpuExecutor, Request, Scheduler
    announce("batch regions sigma %g h %g" % (sigma, h))
    n = 52
    origin = (-0.5 * (n - 1) * h, -0.5 * (n - 1) * h, 3e-3)
    rng = np.random.default_rng(6)
    vol = torch.tensor(rng.uniform(-0.3, 1.0, (n, n, n)).astype(np.float32), device="cuda:0")
    grid, samp = L.Grid(n, n, n, origin, h), L.Sampling(1540.0, 40e6, 512, sigma)
    reqs = []
    for rid, (kind, box, M, K) in enumerate([(POSE, (0, 3, 1, 33, 17, 51), 70, 500), (VOLUME, (5, 0, 9, 16, 31, 25), 64, 400),
                                             (POSE, (7, 7, 7, 9, 25, 37), 5, 300), (VOLUME, (1, 2, 3, 8, 9, 17), 130, 512),
                                             (VOLUME, (0, 0, 0, 20, 8, 48), 64, 512)]):
        pose6 = np.array([0.02, -0.01, 0.3, 1e-4, -2e-4, -3e-3])
        reqs.append(Request(rid, kind, box, W.linear_array(M, 3e-4), pose6, rng.normal(0, 1e-2, (M, K)).astype(np.float32), 2))
    ex = GpuExecutor(vol, grid, samp, slots=6, arena_bytes=1 << 28, graph=False, apply_updates=False)
    sch = Scheduler(ex, 6, 1 << 40)
    for r in reqs:
        sch.submit(r)
    sch.tick()
    assert (ex.info0.rz, ex.info0.moment) == (rz, moment) and len(ex.state) == len(reqs)
    for st in ex.state.values():
        r = st["req"]
        i0, j0, k0, nx, ny, nz = r.box
        bg = L.Grid(nx, ny, nz, (origin[0] + i0 * h, origin[1] + j0 * h, origin[2] + k0 * h), h)
        s = L.Sampling(1540.0, 40e6, r.K, sigma)
        p6 = torch.tensor(r.pose6[None], device="cuda:0")
        gp0 = torch.empty((nx, ny, nz), device="cuda:0")
        gpose = torch.empty((1, 12), dtype=torch.float64, device="cuda:0")
        loss = L.loss_and_grad(bg, vol[i0:i0 + nx, j0:j0 + ny, k0:k0 + nz].contiguous(),
                               torch.tensor(r.elem, device="cuda:0"), L.pose_from_axis_angle(p6), s,
                               torch.tensor(r.y[None], device="cuda:0"), grad_p0=gp0, grad_pose=gpose)
        assert abs(st["losses"][0] - loss) <= 2e-6 * loss
        if r.kind == POSE:
            g6 = L.pose_grad_axis_angle(p6, gpose)[0].cpu().numpy()
            assert rel_l2(st["adam"].cpu().numpy()[:6] / 0.1, g6) <= 1e-5
        else:
            assert rel_l2(st["grad"].cpu().numpy(), gp0.cpu().numpy()) <= 2e-6


def batch_ms(h, sigma=1e-4, n=96, M=128, steps=8):
    import torch
    from paper_2604_09643_amd import _lib as L
    from paper_2604_09643_amd.serve import POSE, VOLUME, GpuExecutor, Request, Scheduler
    rng = np.random.default_rng(5)
    vol = torch.tensor(rng.uniform(-0.3, 1.0, (n, n, n)).astype(np.float32), device="cuda:0")
    grid, samp = L.Grid(n, n, n, (-0.5 * (n - 1) * h, -0.5 * (n - 1) * h, 3e-3), h), L.Sampling(1540.0, 40e6, 1024, sigma)
    ex = GpuExecutor(vol, grid, samp, slots=4, arena_bytes=1 << 30, graph=False, apply_updates=False)
    sch = Scheduler(ex, 4, 1 << 40)
    for rid in range(4):
        sch.submit(Request(rid, POSE if rid % 2 else VOLUME, (0, 0, 0, n, n, n), W.linear_array(M, 3e-4),
                           np.array([0.02, -0.01, 0.3, 1e-4, -2e-4, -3e-3]), rng.normal(0, 1e-2, (M, 1024)).astype(np.float32), steps))
    t = []
    sch.tick()
    while sch.active:
        torch.cuda.synchronize()
        a = time.perf_counter()
        sch.tick()
        t.append(time.perf_counter() - a)
    return sorted(t[:-1])[len(t) // 2 - 1] * 1e3


def test_fine_batches_take_the_moment_forms():
    """Regions of 16 voxels along z below 0.06 mm: as many pairs as on 8; in row form a step took 4 times as long."""
    announce("batch spacings")
    fine, other = batch_ms(5e-5), batch_ms(6e-5)
    assert fine <= 1.6 * other, (fine, other)
