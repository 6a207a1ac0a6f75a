"""The moment-form forward against the FP64 oracle where its split can go wrong: remainders of its regions and
element chunks, each number of moments, both workgroup sizes, records that cut windows, non-finite values."""
import numpy as np
import pytest

from gpu_helpers import announce, gpu_desc, oracle_desc, rel_l2, to_gpu
from oracle import oracle as O
from paper_2604_09643_amd import workloads as W

pytestmark = pytest.mark.gpu

# series 2e-7 and window tails 1.5e-7 of the peak, distance within 4e-6 of half a sample (a slope of about 0.3 peaks
# a sample: 1.2e-6), sums 1.2e-7 and atomic adds a few 1e-7
TOL = 2.5e-6


def forward(w, p0=None, sums=None, static=False):
    import torch
    from paper_2604_09643_amd import _lib as L
    g, s = gpu_desc(w)
    p, elem, poses = to_gpu(w)
    if p0 is not None:
        p = torch.tensor(p0.astype(np.float32), device="cuda:0")
    ctx = L.Context(0)
    if sums is not None:
        ctx.set_forward_sums(sums)
    out = torch.full((w.F, w.M, w.K), 7.0, dtype=torch.float32, device="cuda:0")
    (L.radiate_forward_static if static else L.radiate_forward)(g, p, elem, poses, s, s=out, ctx=ctx)
    got = out.cpu().numpy().astype(np.float64)
    ctx.close()
    return got


def reference(w, p0=None):
    og, os_ = oracle_desc(w)
    p = (w.p0 if p0 is None else p0).astype(np.float32).astype(np.float64)
    return O.grid_forward(og, p, w.poses, w.elem, os_)


@pytest.mark.parametrize("shape,h,M,F,sigma", [
    ((1, 1, 1), 0.1, 1, 1, 0.08), ((3, 2, 7), 0.1, 3, 1, 0.08), ((5, 4, 8), 0.2, 64, 1, 0.1),
    ((16, 16, 16), 0.1, 13, 5, 0.08), ((17, 15, 9), 0.1, 65, 1, 0.12), ((33, 18, 17), 0.1, 63, 2, 0.1),
    ((18, 35, 23), 0.08, 43, 3, 0.08), ((20, 9, 40), 0.05, 16, 4, 0.06), ((9, 8, 30), 0.2, 33, 2, 0.055),
    ((16, 7, 24), 0.125, 32, 4, 0.04)])
def test_shapes(shape, h, M, F, sigma):
    announce("moment forward %s h %g M %d F %d sigma %g" % (shape, h, M, F, sigma))
    w = W.small(shape=shape, h=h * 1e-3, M=M, F=F, K=700, sigma=sigma * 1e-3)
    ref = reference(w)
    assert rel_l2(forward(w), ref) <= TOL
    assert rel_l2(forward(w, sums=2), ref) <= TOL
    assert rel_l2(forward(w, static=True), ref) <= TOL


@pytest.mark.parametrize("K", [1, 40, 180, 230])
def test_record_cuts_windows(K):
    announce("moment forward K %d" % K)
    w = W.small(shape=(17, 12, 20), h=1e-4, M=70, F=1, K=K, sigma=8e-5)
    ref = reference(w)
    got = forward(w)
    if np.abs(ref).max() == 0.0:
        assert np.all(got == 0.0)
    else:
        assert rel_l2(got, ref) <= TOL


@pytest.mark.parametrize("scale", [1e-20, 1e15])
def test_scale_of_p0(scale):
    announce("moment forward scale %g" % scale)
    w = W.small(shape=(18, 12, 20), h=1e-4, M=20, F=2, K=500, sigma=8e-5)
    assert rel_l2(forward(w, w.p0 * scale), reference(w, w.p0 * scale)) <= TOL


def test_one_bright_voxel_and_zeros():
    announce("moment forward sparse")
    w = W.small(shape=(34, 20, 20), h=1e-4, M=20, F=2, K=500, sigma=8e-5)
    p = np.zeros(w.shape)
    assert np.all(forward(w, p) == 0.0)
    p[20, 3, 19] = -3.0
    p[2, 3, 4] = 1e-3
    assert rel_l2(forward(w, p), reference(w, p)) <= TOL


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_non_finite_p0_reaches_its_window_and_no_more(bad):
    announce("moment forward p0 %g" % bad)
    w = W.small(shape=(18, 12, 20), h=1e-4, M=20, F=2, K=500, sigma=8e-5)
    p = w.p0.copy()
    p[3, 4, 5] = bad
    q = np.zeros(w.shape)
    q[3, 4, 5] = 1.0
    got, ref, mark = forward(w, p), reference(w, w.p0), reference(w, q)
    hit = mark != 0.0
    assert not np.isfinite(got[hit]).any()
    # rows are taken whole: at most one sample past the window on either side
    near = hit.copy()
    near[..., 1:] |= hit[..., :-1]
    near[..., :-1] |= hit[..., 1:]
    assert np.isfinite(got[~near]).all()
    q[3, 4, 5] = w.p0[3, 4, 5]
    far = ~near
    assert rel_l2(got[far], ref[far]) <= TOL


def test_non_finite_pose_stays_in_its_frame():
    announce("moment forward NaN pose")
    w = W.small(shape=(18, 12, 20), h=1e-4, M=70, F=2, K=500, sigma=8e-5)
    ref = reference(w)
    w.poses = w.poses.copy()
    w.poses[1, 9] = np.nan
    got = forward(w)
    assert rel_l2(got[0], ref[0]) <= TOL
    assert not np.isfinite(got[1]).all()


def test_elements_close_to_and_inside_the_grid():
    """Nearer than the far-field model allows: the values still follow the formula."""
    announce("moment forward near elements")
    w = W.small(shape=(17, 12, 20), h=1e-4, M=5, F=1, K=200, sigma=8e-5)
    z0 = w.origin[2]
    w.elem = np.array([[0.0, 0.0, z0 - 3e-4], [3.3e-4, 1e-5, z0 - 6e-5], [1.2e-4, 4e-5, z0 + 4.31e-4],
                       [0.0, 0.0, z0 - 2e-3], [5e-3, 0.0, z0]])
    w.poses = np.array([[1.0, 0, 0, 0, 1.0, 0, 0, 0, 1.0, 0, 0, 0]])
    got, ref = forward(w), reference(w)
    for m in range(5):
        assert rel_l2(got[0, m], ref[0, m]) <= 1e-5
