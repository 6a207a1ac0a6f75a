"""The context keeps the series of the samplings used last: a program that alternates widths pays for none again."""
import time

import pytest

from gpu_helpers import announce
from paper_2604_09643_amd import workloads as W

pytestmark = pytest.mark.gpu


def loop_us(f, runs=9):
    import torch
    f()
    t = []
    for _ in range(runs):
        torch.cuda.synchronize()
        a = time.perf_counter()
        f()
        torch.cuda.synchronize()
        t.append(time.perf_counter() - a)
    return sorted(t)[runs // 2] * 1e6


def test_alternating_samplings_cost_what_one_does():
    import torch
    from paper_2604_09643_amd import _lib as L
    announce("alternating samplings")
    g = L.Grid(8, 8, 8, (0.0, 0.0, 6e-3), 1e-4)
    dev = "cuda:0"
    p = torch.randn((8, 8, 8), device=dev)
    elem = torch.tensor(W.linear_array(16, 3e-4), dtype=torch.float64, device=dev)
    poses = torch.tensor([[1.0, 0, 0, 0, 1.0, 0, 0, 0, 1.0, 0, 0, 0]], dtype=torch.float64, device=dev)
    every = [L.Sampling(1540.0, 40e6, 512, sg) for sg in (1e-4, 9e-5, 8e-5)]
    out = torch.empty((1, 16, 512), device=dev)

    def loop(kinds):
        for i in range(60):
            L.radiate_forward(g, p, elem, poses, kinds[i % len(kinds)], s=out)
    one, three = loop_us(lambda: loop(every[:1])), loop_us(lambda: loop(every))
    assert three <= 1.25 * one, (one / 60, three / 60)      # 21 and 31 us a call where the last series alone is kept
