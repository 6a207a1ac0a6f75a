"""Volumes whose voxels differ by many orders of magnitude inside one region: what the bright ones do not reach keeps
its digits.  Signals against the FP64 oracle, at the samples outside the bright voxels' windows alone."""
import numpy as np
import pytest

from gpu_helpers import announce, gpu_desc, oracle_desc, rel_l2, to_gpu
from oracle import oracle as O
from paper_2604_09643_amd import workloads as W

pytestmark = pytest.mark.gpu

# as for volumes of like voxels: the Gaussian's series and window tails 2e-7, distance 1.2e-6, sums a few 1e-7; the
# power law's long windows 1e-5.  In one class with the bright voxels a term is rounded to 2^-17 of its line's largest
TOL, TOL_ONE = 2.5e-6, 1e-5


def pattern(name, shape, rng):
    p = 0.01 * rng.normal(size=shape)
    m = np.zeros(shape, dtype=bool)
    if name == "voxel":
        m[3, 4, 5] = True
    elif name == "plane":
        m[:, :, 6] = True
    elif name == "scattered":
        m = rng.random(shape) < 0.01
    elif name == "three":                  # three magnitudes
        p[10:] *= 1e5
        m[15, 15, 15] = True
    return p, m


@pytest.mark.parametrize("kernel,trunc", [(0, 6.0), (2, 10.0)])
@pytest.mark.parametrize("name,value,tol", [("voxel", 1e4, TOL), ("voxel", 1e8, TOL), ("plane", 1e6, TOL), ("scattered", -1e5, TOL),
                                            ("three", 1e9, TOL), ("voxel", 30.0, TOL_ONE)])
def test_faint_voxels_keep_their_digits(name, value, tol, kernel, trunc):
    import torch
    from paper_2604_09643_amd import _lib as L
    announce("classes %s %g kernel %d" % (name, value, kernel))
    w = W.small(shape=(16, 16, 16), h=1e-4, M=70, F=1, K=500, sigma=8e-5)
    rng = np.random.default_rng(11)
    p, bright = pattern(name, w.shape, rng)
    p[bright] = value
    w.p0 = p
    (g, _), (pt, elem, poses) = gpu_desc(w), to_gpu(w)
    s = L.Sampling(w.c, w.fs, w.K, w.sigma, trunc, kernel, 2.0)
    got = L.radiate_forward(g, pt, elem, poses, s).cpu().numpy()
    og, os_ = oracle_desc(w)[0], O.Sampling(w.c, w.fs, w.K, w.sigma, trunc, kernel, 2.0)
    p32 = p.astype(np.float32).astype(np.float64)
    ref = O.grid_forward(og, p32, w.poses, w.elem, os_)
    reach = O.grid_forward(og, bright.astype(np.float64), w.poses, w.elem, O.Sampling(w.c, w.fs, w.K, w.sigma, trunc + 1.0, kernel, 2.0))
    far = reach == 0.0                     # rows are taken whole, half a sample past the window: one width is more
    assert (np.abs(ref[far]) > 0.0).sum() > 300
    tol = max(tol, 1e-5) if kernel else tol
    assert rel_l2(got, ref) <= tol
    if name == "three":                    # and where only the faintest reach
        far &= O.grid_forward(og, (np.abs(p) > 1.0).astype(np.float64), w.poses, w.elem, O.Sampling(
            w.c, w.fs, w.K, w.sigma, trunc + 1.0, kernel, 2.0)) == 0.0
    assert rel_l2(got[far], ref[far]) <= tol
