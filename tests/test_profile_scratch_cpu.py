"""Scratch of the power-law, exponential and narrow Gaussian calls: the moment table (up to 48 bytes per sample) is part of it for ordinary
sweeps and left out where it would exceed 16 GiB, so that large sweeps need what the row forms need."""
import ctypes

import pytest

from paper_2604_09643_amd import _lib as L


@pytest.mark.parametrize("kernel,nu,trunc,width", [(1, 1.0, 12.0, 8e-5), (2, 2.0, 10.0, 8e-5), (0, 1.0, 6.0, 6.5e-5)])
def test_table_is_bounded(kernel, nu, trunc, width):
    lib = L.load()
    g = L.Grid(16, 16, 16, (0.0, 0.0, 0.05), 1e-4)
    K, jt = 2048, 22
    s = L.Sampling(1540.0, 40e6, K, width, trunc, kernel, nu)
    for F, rows in ((4, True), (260, False)):         # rows: of the moment table
        E = 4096 * F
        n = lib.ra_scratch_bytes(ctypes.byref(g.c()), 4096, F, ctypes.byref(s.cs()))
        # signals in FP32 and FP64, element data, and the partials of at most 64 regions
        plain = E * K * 12 + E * 64 * 24 + E * 100 + (1 << 20)
        assert (n > plain) == rows, (F, n, plain)
        assert n <= plain + min(16 << 30, E * (K + 2 * jt + 10) * 48)
