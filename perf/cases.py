"""Workloads of the radiation library for timing and for comparing two builds of it.

Each case is one call, or one short loop of calls, that a program using this framework makes:
simulating signals, reconstructing a volume, refining poses, localising elements, regularising
a volume, serving requests.  Sizes follow the configurations of `workloads.py`, the tests and
`bench.py`; `draw` spreads them, odd sizes included, over the ranges those cover.

Volumes hold vessel-like tubes over a low background, as a reconstruction in progress does.
Signals given as measurements are band-limited noise of the amplitude the forward model
produces for such a volume.  Poses and scores leave a pass in float32, the type a tracking
program hands on.
"""
import math

import numpy as np
import torch

from paper_2604_09643_amd import _lib as L
from paper_2604_09643_amd import autograd as A
from paper_2604_09643_amd import localise, rigid, serve
from paper_2604_09643_amd import workloads as W

MM = 1e-3
GAUSS, EXPONENTIAL, POWER, UNIFORM = range(4)
EXACT_MOST = 1.0e11          # (voxel, element, sample) terms up to which `exact` sums them one by one

_BASE = {"op": "forward", "nx": 32, "ny": 32, "nz": 32, "h_um": 100.0, "depth_mm": 6.0, "array": "line", "M": 64,
         "F": 1, "K": 1024, "sigma_um": 80.0, "kernel": GAUSS, "trunc": 6.0, "nu": 2.0, "chunk": 16, "steps": 1,
         "N": 0}


def _case(name=None, **kw):
    c = dict(_BASE)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one frame of a 64-element probe on a small box: the smallest call, made per frame in a tracking loop
        _case("preview_forward", op="forward", nx=32, ny=32, nz=32, h_um=200.0, K=512, sigma_um=100.0),
        # the single freehand sweep: one data-term step of a reconstruction (the benchmark's own step)
        _case("sweep_loss_grad", op="loss", nx=128, ny=128, nz=64, depth_mm=6.85, M=128, F=64, K=1024),
        # joint reconstruction and pose refinement of a short sweep on a ragged grid: loss, backward to both
        _case("joint_sweep_step", op="sweep", nx=97, ny=101, nz=59, h_um=80.0, M=96, F=11, K=1000, chunk=4),
        # a volume seen by a 32 x 32 matrix array: signals and their backward to volume and pose
        _case("matrix_radiate", op="radiate", nx=192, ny=192, nz=192, depth_mm=2.0, array="matrix", M=1024, F=1,
              K=2048, sigma_um=100.0),
        # simulated signals of one 512-element view of the hemispherical array
        _case("hemisphere_forward", op="forward", nx=224, ny=224, nz=160, array="cap", M=512, F=1, K=2560,
              sigma_um=100.0),
        # back-projection alone: the volume gradient of given residuals, sparse 33-element cap, three views
        _case("cap_backproject", op="adjoint", nx=161, ny=147, nz=130, array="cap33", M=33, F=3, K=2048,
              sigma_um=100.0),
        # element localisation: scores of lattice candidates against one measured row each
        _case("localise_scores", op="scores", nx=48, ny=48, nz=40, M=1, N=3000, K=1024, sigma_um=120.0),
        # pose fine-tuning: four optimiser steps on one 64-element frame
        _case("finetune_pose", op="finetune", nx=72, ny=64, nz=64, M=64, K=1024, steps=4),
        # another source profile, smooth with a long tail: one data-term step
        _case("power_loss_grad", op="loss", nx=64, ny=60, nz=48, M=64, F=6, K=1024, kernel=POWER, trunc=10.0),
        # another source profile, exponential: one data-term step
        _case("exponential_loss_grad", op="loss", nx=64, ny=60, nz=48, M=64, F=6, K=1024, kernel=EXPONENTIAL,
              trunc=12.0),
        # the regulariser of a reconstruction step on a full volume
        _case("tgv_step", op="tgv", nx=256, ny=256, nz=256),
        # request stream: poses and volume updates of mixed sizes through the batching loop
        _case("serve_mixed", op="serve", nx=192, ny=192, nz=192, depth_mm=2.0, N=6, steps=3, sigma_um=100.0),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _pairs(c):
    return float(c["nx"]) * c["ny"] * c["nz"] * c["M"] * c["F"]


def draw(rng):
    """One more case of the same ranges.  Boxes of 16 to 256 voxels a side, arrays of 16 to 1024
    elements, 1 to 64 frames, kernel widths 0.06 to 0.125 mm."""
    op = rng.choice(["forward", "forward", "loss", "loss", "adjoint", "radiate", "sweep", "scores", "finetune", "tgv",
                     "serve"])
    side = lambda lo, hi: int(round(_log(rng, lo, hi)))  # noqa: E731
    K = rng.choice([512, 777, 1000, 1024, 1536, 2048])
    c = _case(op=op, sigma_um=round(rng.uniform(60.0, 125.0), 1), K=K, depth_mm=round(rng.uniform(3.0, 8.0), 2),
              h_um=rng.choice([80.0, 100.0, 100.0, 125.0, 200.0]))
    if op == "tgv":
        c.update(nx=side(24, 256), ny=side(24, 256), nz=side(24, 256))
        return c
    if op == "serve":
        n = side(96, 192)
        c.update(nx=n, ny=n, nz=n, h_um=100.0, depth_mm=2.0, N=rng.randint(1, 6), steps=rng.randint(1, 3),
                 sigma_um=round(rng.uniform(80.0, 110.0), 1))
        return c
    if op == "scores":
        c.update(nx=side(24, 64), ny=side(24, 64), nz=side(24, 64), M=1, N=side(64, 3000))
        return c
    if op == "finetune":
        c.update(nx=side(32, 96), ny=side(32, 96), nz=side(32, 96), M=side(16, 128), steps=rng.randint(1, 4))
        return c
    kind = rng.choice(["line", "line", "matrix", "cap33"])
    M = {"line": rng.choice([32, 48, 64, 96, 128, 130]), "matrix": rng.choice([64, 256, 576]), "cap33": 33}[kind]
    c.update(array=kind, M=M, F=side(1, 24))
    if op in ("forward", "loss") and rng.random() < 0.4:
        c["kernel"] = rng.choice([EXPONENTIAL, POWER, UNIFORM])
        c["trunc"] = {EXPONENTIAL: 12.0, POWER: 10.0, UNIFORM: 1.0}[c["kernel"]]
        c["nu"] = rng.choice([1.5, 2.0, 2.0, 3.0])
        c["sigma_um"] = round(rng.uniform(60.0, 100.0), 1)
    # the volume takes what is left of the largest listed step (a tenth of it for the other profiles)
    most = 8.0e9 if c["kernel"] == GAUSS else 5.0e8
    c.update(nx=side(16, 200), ny=side(16, 200), nz=side(16, 160))
    while _pairs(c) > most:
        if c["F"] > 1:
            c["F"] = max(1, c["F"] // 2)
        else:
            c.update(nx=max(16, c["nx"] // 2 + 1), ny=max(16, c["ny"] // 2 + 1))
    c["chunk"] = rng.choice([3, 4, 16])
    return c


# ----------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------

def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _shape(c):
    return (c["nx"], c["ny"], c["nz"])


def _origin(c):
    """Corner voxel of the box: centred at the origin for the caps, else centred under the array."""
    h = c["h_um"] * 1e-6
    o = [-0.5 * (n - 1) * h for n in _shape(c)]
    if not c["array"].startswith("cap"):
        o[2] = c["depth_mm"] * MM
    return tuple(o)


def _elements(c):
    if c["array"] == "matrix":
        return W.matrix_array(int(round(math.sqrt(c["M"]))), 0.5 * MM)
    if c["array"] == "cap":
        full = W.fibonacci_cap(2 * c["M"], 60 * MM, np.pi / 2)
        order = np.argsort(np.mod(np.arctan2(full[:, 1], full[:, 0]), 2 * np.pi), kind="stable")
        return full[np.sort(order[:c["M"]])]
    if c["array"] == "cap33":
        return W.fibonacci_cap(c["M"], 40 * MM, np.deg2rad(35.0))
    return W.linear_array(c["M"], 0.3 * MM)


def _pose6(c, rng):
    return W.sweep_pose6(c["F"], 0.1 * MM, 0.2 * MM, 1.0, rng)


def _volume(c, seed, device):
    """Tubes along random walks (values 0.3 to 1) over a background of standard deviation 0.01."""
    g = torch.Generator().manual_seed(int(seed) * 7 + 1)
    shape = torch.tensor(_shape(c), dtype=torch.float64)
    vol = torch.zeros(_shape(c), dtype=torch.float32, device=device)
    for _ in range(12):
        p = (0.1 + 0.8 * torch.rand(3, generator=g, dtype=torch.float64)) * (shape - 1)
        v = torch.randn(3, generator=g, dtype=torch.float64)
        r = 1.0 + 4.0 * float(torch.rand(1, generator=g))
        value = 0.3 + 0.7 * float(torch.rand(1, generator=g))
        for _ in range(24):
            v = v + 0.4 * torch.randn(3, generator=g, dtype=torch.float64)
            v = v / v.norm()
            p = torch.minimum(torch.maximum(p + r * v, torch.zeros(3, dtype=torch.float64)), shape - 1)
            lo = [max(0, int(math.floor(float(p[a]) - r))) for a in range(3)]
            hi = [min(_shape(c)[a], int(math.ceil(float(p[a]) + r)) + 1) for a in range(3)]
            ax = [torch.arange(lo[a], hi[a], device=device, dtype=torch.float32) - float(p[a]) for a in range(3)]
            inside = ax[0][:, None, None] ** 2 + ax[1][None, :, None] ** 2 + ax[2][None, None, :] ** 2 <= r * r
            sub = vol[lo[0]:hi[0], lo[1]:hi[1], lo[2]:hi[2]]
            sub.copy_(torch.maximum(sub, value * inside.to(torch.float32)))
    gd = torch.Generator(device=device).manual_seed(int(seed) * 7 + 2)
    return vol + 0.01 * torch.randn(vol.shape, generator=gd, device=device)


def _signals(rows, K, seed, device, scale):
    """Band-limited noise, one row an element."""
    g = torch.Generator(device=device).manual_seed(int(seed) * 7 + 3)
    x = torch.randn((rows, K + 8), generator=g, device=device)
    x = x.unfold(1, 9, 1).mean(-1) * 3.0
    return (scale * x).contiguous()


def _scale(c):
    """About half the rms of the signals of such a volume: a shell crosses the box in nx ny voxels'
    worth of area per spacing, each adding a zero-mean pulse of width sigma."""
    d = 40 * MM if c["array"].startswith("cap") else (c["depth_mm"] + 3.0) * MM
    shell = math.sqrt(c["nx"] * c["ny"] * c["sigma_um"] / c["h_um"])
    return 0.1 * c["sigma_um"] * 1e-6 / (2 * d) * shell


def _inputs(c, seed, device):
    rng = np.random.default_rng(int(seed) * 7 + 4)
    pose6 = torch.tensor(_pose6(c, rng), dtype=torch.float64, device=device)
    elem = torch.tensor(_elements(c), dtype=torch.float64, device=device).contiguous()
    return {"p0": _volume(c, seed, device), "elem": elem, "pose6": pose6}


def _poses(pose6):
    p = W.poses_from_pose6(pose6.cpu().numpy())
    return torch.tensor(p, dtype=torch.float64, device=pose6.device)


def _candidates(c, seed, device):
    """Lattice-like candidate positions above the box, within 3 mm of a guess."""
    rng = np.random.default_rng(int(seed) * 7 + 5)
    return torch.tensor(rng.uniform(-1.5, 1.5, size=(c["N"], 3)) * MM, dtype=torch.float64, device=device)


def prepare(case, seed):
    c, dev = case, _dev()
    st = {"c": c, "grid": L.Grid(*_shape(c), _origin(c), c["h_um"] * 1e-6),
          "samp": L.Sampling(W.C_SOUND, W.FS, c["K"], c["sigma_um"] * 1e-6, c["trunc"], c["kernel"], c["nu"])}
    op, K = c["op"], c["K"]
    if op == "tgv":
        u = _volume(c, seed, dev)
        g = torch.Generator(device=dev).manual_seed(int(seed) * 7 + 6)
        st.update(u=u, w=0.02 * torch.randn((3,) + _shape(c), generator=g, device=dev), gu=torch.empty_like(u),
                  gw=torch.empty((3,) + _shape(c), device=dev))
        return st
    if op == "serve":
        vol = _volume(c, seed, dev)
        st["ex"] = serve.GpuExecutor(vol, st["grid"], st["samp"], slots=8, arena_bytes=1 << 30, apply_updates=False)
        # the mix of the requests (kinds, arrays, boxes) belongs to the case, poses and signals to the seed
        side = (min(48, c["nx"]), min(128, c["nx"]))
        specs = W.serving_stream(c["N"], 1e3, _shape(c), _origin(c), c["h_um"] * 1e-6, seed=c["N"], side=side,
                                 Ks=(512, 1024), pose_steps=c["steps"])
        rng = np.random.default_rng(int(seed) * 7 + 9)
        jitter = [np.concatenate([rng.normal(0, 0.01, 3), rng.normal(0, 0.1 * MM, 3)]) for _ in specs]
        st["specs"] = [(s, s.true6 + d, _signals(s.M, s.K, 31 * int(seed) + s.rid, dev, _scale(c)).cpu().numpy())
                       for s, d in zip(specs, jitter)]
        return st
    st.update(_inputs(c, seed, dev))
    E = c["F"] * c["M"]
    if op == "forward":
        st["poses"] = _poses(st["pose6"])
    elif op == "loss":
        st.update(poses=_poses(st["pose6"]), y=_signals(E, K, seed, dev, _scale(c)).view(c["F"], c["M"], K),
                  gp0=torch.empty_like(st["p0"]))
    elif op == "adjoint":
        st.update(poses=_poses(st["pose6"]), r=_signals(E, K, seed, dev, 1.0).view(c["F"], c["M"], K),
                  gp0=torch.empty_like(st["p0"]))
    elif op == "radiate":
        st["gs"] = _signals(E, K, seed, dev, 1.0).view(c["F"], c["M"], K)
        st["pose32"] = st["pose6"].float()
    elif op == "sweep":
        st["y"] = _signals(E, K, seed, dev, _scale(c)).view(c["F"], c["M"], K)
        st["pose32"] = st["pose6"].float()
    elif op == "scores":
        st.update(cand=_candidates(c, seed, dev), y=_signals(c["N"], K, seed, dev, _scale(c)))
    elif op == "finetune":
        rng = np.random.default_rng(int(seed) * 7 + 8)
        st.update(y=_signals(c["M"], K, seed, dev, _scale(c)), inliers=(rng.random(c["M"]) < 0.85).astype(np.float32),
                  euler6=np.concatenate([rng.normal(0, 0.02, 3), rng.normal(0, 0.2 * MM, 3)]),
                  template=_elements(c))
    return st


# ----------------------------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------------------------

def _leaves(st):
    return st["p0"].detach().requires_grad_(True), st["pose32"].detach().requires_grad_(True)


def run(st):
    c, op = st["c"], st["c"]["op"]
    if op == "forward":
        return L.radiate_forward(st["grid"], st["p0"], st["elem"], st["poses"], st["samp"])
    if op == "loss":
        loss = L.loss_and_grad(st["grid"], st["p0"], st["elem"], st["poses"], st["samp"], st["y"], grad_p0=st["gp0"])
        return {"loss": loss, "grad_p0": st["gp0"]}
    if op == "adjoint":
        L.radiate_adjoint(st["grid"], None, st["elem"], st["poses"], st["samp"], st["r"], grad_p0=st["gp0"])
        return {"grad_p0": st["gp0"]}
    if op == "radiate":
        p, w = _leaves(st)
        s = A.radiate(p, w.double(), st["elem"], st["grid"], st["samp"])
        s.backward(st["gs"])
        return {"s": s.detach(), "grad_p0": p.grad, "grad_pose": w.grad}
    if op == "sweep":
        p, w = _leaves(st)
        loss = A.sweep_loss(p, w.double(), st["y"], st["elem"], st["grid"], st["samp"], chunk=c["chunk"])
        loss.backward()
        return {"loss": loss.detach().float(), "grad_p0": p.grad, "grad_pose": w.grad}
    if op == "scores":
        s = localise.nc_scores(st["grid"], st["p0"], st["samp"], st["y"], st["cand"])
        return {"scores": s.astype(np.float32)}
    if op == "finetune":
        hist = []
        p6 = rigid.finetune(st["grid"], st["p0"], st["samp"], st["y"], st["template"], st["euler6"], st["inliers"],
                            steps=c["steps"], history=hist)
        return {"pose": p6.float(), "losses": hist}
    if op == "tgv":
        v = L.tgv_loss_and_grad(st["u"], st["w"], 2.0, 1.0, 1e-3, scale=0.1, grad_u=st["gu"], grad_w=st["gw"])
        return {"value": v, "grad_u": st["gu"], "grad_w": st["gw"]}
    reqs = [serve.Request(s.rid, s.kind, s.box, s.elem, pose6, y, s.steps) for s, pose6, y in st["specs"]]
    _, results = serve.serve(st["ex"], reqs, 8, 1 << 30, realtime=False)
    out = {}
    for r in results:
        out["r%02d" % r.rid] = {"losses": r.losses, "grad": r.grad_p0,
                                "pose": None if r.pose6 is None else r.pose6.astype(np.float32)}
    return out


# ----------------------------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------------------------

def work(case):
    """Inputs read once, outputs written once.  Operations: a (voxel, element) pair needs at least its
    distance (10), its place in the record (4) and one pass over an 8-coefficient local expansion of
    the pulse (16), each way; the expansion of a row into samples and the statistics are small."""
    c = case
    nv = float(c["nx"]) * c["ny"] * c["nz"]
    if c["op"] == "tgv":
        return {"bytes": 32.0 * nv, "flops": 150.0 * nv}
    if c["op"] == "serve":
        vox = 88.0 ** 3
        return {"bytes": c["N"] * 8.0 * vox, "flops": c["N"] * (0.7 * c["steps"] + 0.3) * 150 * vox * 60.0}
    E = c["N"] if c["op"] == "scores" else c["F"] * c["M"]
    ways = {"forward": 1, "adjoint": 1, "scores": 1, "loss": 2, "radiate": 2.5, "sweep": 2.5,
            "finetune": 2.5 * c["steps"]}[c["op"]]
    rows = {"forward": 1, "adjoint": 1, "scores": 1, "loss": 1, "radiate": 2, "sweep": 1, "finetune": 1}[c["op"]]
    vols = {"forward": 1, "adjoint": 1, "scores": 1, "finetune": 1}.get(c["op"], 2)
    return {"bytes": 4.0 * (vols * nv + rows * E * c["K"]), "flops": ways * 30.0 * nv * E}


# ----------------------------------------------------------------------------------------------
# the same in 64 bits, term by term
# ----------------------------------------------------------------------------------------------

class _Model:
    """Forward model and adjoints of one geometry in float64: every (voxel, element, sample) term with
    |d - c t_k| <= trunc sigma, one sample offset at a time."""

    def __init__(self, c, device):
        self.c, self.dev = c, device
        h, o = c["h_um"] * 1e-6, _origin(c)
        ax = [torch.arange(n, dtype=torch.float64, device=device) * h + o[a] for a, n in enumerate(_shape(c))]
        self.x = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
        self.delta = W.C_SOUND / W.FS
        self.w = c["sigma_um"] * 1e-6
        self.tsig = c["trunc"] * self.w
        self.J = int(math.floor(self.tsig / self.delta + 0.5))

    def phi(self, u):
        k, a = self.c["kernel"], u.abs()
        if k == GAUSS:
            return u * torch.exp(-0.5 * (u / self.w) ** 2)
        if k == EXPONENTIAL:
            return u * torch.exp(-a / self.w)
        if k == POWER:
            return u * (1 + (u / self.w) ** 2) ** (-self.c["nu"])
        return u

    def dphi(self, u):
        k, a = self.c["kernel"], u.abs()
        if k == GAUSS:
            return (1 - (u / self.w) ** 2) * torch.exp(-0.5 * (u / self.w) ** 2)
        if k == EXPONENTIAL:
            return (1 - a / self.w) * torch.exp(-a / self.w)
        if k == POWER:
            q = (u / self.w) ** 2
            return (1 - 2 * self.c["nu"] * q / (1 + q)) * (1 + q) ** (-self.c["nu"])
        return torch.ones_like(u)

    def _blocks(self, X):
        eb = max(1, int(2 ** 24 // self.x.shape[0]))
        vb = min(self.x.shape[0], 2 ** 24)
        for e0 in range(0, X.shape[0], eb):
            for v0 in range(0, self.x.shape[0], vb):
                xe, xv = X[e0:e0 + eb], self.x[v0:v0 + vb]
                diff2 = sum((xe[:, None, a] - xv[None, :, a]) ** 2 for a in range(3))
                yield slice(e0, e0 + eb), slice(v0, v0 + vb), diff2.sqrt()

    def _terms(self, d):
        k0 = torch.round(d / self.delta)
        for j in range(-self.J, self.J + 1):
            k = k0 + j
            u = d - k * self.delta
            keep = (u.abs() <= self.tsig) & (k >= 0) & (k < self.c["K"])
            yield k.clamp(0, self.c["K"] - 1).long(), u, keep

    def forward(self, p, X):
        """The terms of one sample offset, voxels in the order of their centre sample, add up as differences
        of their running sum."""
        K, J = self.c["K"], self.J
        s = torch.zeros((X.shape[0], K), dtype=torch.float64, device=self.dev)
        for es, vs, d in self._blocks(X):
            k0, order = torch.sort(torch.round(d / self.delta), dim=1)
            d = torch.gather(d, 1, order)
            a = p[vs][order] / (2 * d)
            marks = torch.arange(-J, K + J + 1, dtype=torch.float64, device=self.dev).expand(d.shape[0], -1)
            at = torch.searchsorted(k0.contiguous(), marks.contiguous())      # first voxel of centre sample >= mark
            run = torch.zeros((d.shape[0], d.shape[1] + 1), dtype=torch.float64, device=self.dev)
            for j in range(-J, J + 1):
                u = d - (k0 + j) * self.delta
                torch.cumsum(torch.where(u.abs() <= self.tsig, a * self.phi(u), 0.0), 1, out=run[:, 1:])
                first, last = at[:, J - j:J - j + K], at[:, J - j + 1:J - j + 1 + K]
                s[es] += torch.gather(run, 1, last) - torch.gather(run, 1, first)
        return s

    def adjoint(self, p, X, r, want_p0=True, want_x=False):
        gp = torch.zeros(self.x.shape[0], dtype=torch.float64, device=self.dev) if want_p0 else None
        gx = torch.zeros_like(X) if want_x else None
        for es, vs, d in self._blocks(X):
            Aa, Bb = torch.zeros_like(d), torch.zeros_like(d)
            for k, u, keep in self._terms(d):
                rk = torch.where(keep, torch.gather(r[es], 1, k), 0.0)
                Aa += rk * self.phi(u)
                if want_x:
                    Bb += rk * self.dphi(u)
            if want_p0:
                gp[vs] += (Aa / (2 * d)).sum(0)
            if want_x:
                coef = p[vs][None] * (Bb / (2 * d) - Aa / (2 * d * d)) / d
                gx[es] += X[es] * coef.sum(1, keepdim=True) - coef @ self.x[vs]
        return gp, gx


def _rotation(w):
    """Rotation matrices of axis-angle vectors [F, 3], differentiable."""
    z = torch.zeros_like(w[:, 0])
    k = torch.stack([z, -w[:, 2], w[:, 1], w[:, 2], z, -w[:, 0], -w[:, 1], w[:, 0], z], -1).reshape(-1, 3, 3)
    return torch.matrix_exp(k)


def _place(pose6, elem):
    R = _rotation(pose6[:, :3])
    return ((R[:, None] * elem[None, :, None, :]).sum(-1) + pose6[:, None, 3:]).reshape(-1, 3)


def _nc(s, y):
    """Negative correlation of each row and its gradient with respect to s."""
    K = s.shape[1]
    ds, dy = s - s.mean(1, keepdim=True), y - y.mean(1, keepdim=True)
    C = (ds * dy).mean(1, keepdim=True)
    ss, sy = (ds * ds).mean(1, keepdim=True).sqrt(), (dy * dy).mean(1, keepdim=True).sqrt()
    return -(C / (ss * sy))[:, 0], -dy / (K * ss * sy) + C * ds / (K * ss ** 3 * sy)


def exact(case, seed):
    c, op, dev = case, case["op"], _dev()
    if op == "serve":
        return None              # a whole engine
    if op == "tgv":
        if c["nx"] * c["ny"] * c["nz"] > 2 ** 24:
            return None
        g = torch.Generator(device=dev).manual_seed(int(seed) * 7 + 6)
        w = (0.02 * torch.randn((3,) + _shape(c), generator=g, device=dev)).double()
        return _exact_tgv(_volume(c, seed, dev).double(), w)
    m = _Model(c, dev)
    E = c["N"] if op == "scores" else c["F"] * c["M"]
    passes = {"forward": 1, "adjoint": 1, "scores": 1, "finetune": 2 * c["steps"]}.get(op, 2)
    if m.x.shape[0] * float(E) * (2 * m.J + 1) * passes > EXACT_MOST:
        return None
    i = _inputs(c, seed, dev)
    p = i["p0"].double().reshape(-1)
    K = c["K"]
    if op == "scores":
        X = _candidates(c, seed, dev)
        return {"scores": _nc(m.forward(p, X), _signals(c["N"], K, seed, dev, _scale(c)).double())[0]}
    if op == "finetune":
        return _exact_finetune(c, seed, m, p, i["elem"], dev)
    if op in ("radiate", "sweep"):
        pose = i["pose6"].float().double().requires_grad_(True)
        Xg = _place(pose, i["elem"])
    else:
        Xg = _place(i["pose6"], i["elem"])
    X = Xg.detach()
    if op == "forward":
        return m.forward(p, X).view(c["F"], c["M"], K)
    if op == "adjoint":
        return {"grad_p0": m.adjoint(p, X, _signals(E, K, seed, dev, 1.0).double())[0].view(_shape(c))}
    s = m.forward(p, X)
    if op == "radiate":
        gp, gx = m.adjoint(p, X, _signals(E, K, seed, dev, 1.0).double(), want_x=True)
        Xg.backward(gx)
        return {"s": s.view(c["F"], c["M"], K), "grad_p0": gp.view(_shape(c)), "grad_pose": pose.grad}
    res = s - _signals(E, K, seed, dev, _scale(c)).double()
    gp, gx = m.adjoint(p, X, 2 * res, want_x=op == "sweep")
    out = {"loss": float((res * res).sum()), "grad_p0": gp.view(_shape(c))}
    if op == "sweep":
        Xg.backward(gx)
        out["grad_pose"] = pose.grad
    return out


def _exact_finetune(c, seed, m, p, elem, dev):
    rng = np.random.default_rng(int(seed) * 7 + 8)
    wt = torch.tensor((rng.random(c["M"]) < 0.85).astype(np.float64), device=dev)
    e6 = np.concatenate([rng.normal(0, 0.02, 3), rng.normal(0, 0.2 * MM, 3)])
    y = _signals(c["M"], c["K"], seed, dev, _scale(c)).double()
    a = torch.tensor(e6[:3], device=dev).requires_grad_(True)
    t = torch.tensor(e6[3:], device=dev).requires_grad_(True)
    opt = torch.optim.Adam([{"params": [a], "lr": 1e-3}, {"params": [t], "lr": 1e-5}])
    hist = []
    unit = torch.eye(3, dtype=torch.float64, device=dev)
    for _ in range(c["steps"]):
        opt.zero_grad()
        Rx, Ry, Rz = (_rotation((a[q] * unit[q])[None])[0] for q in range(3))
        R = Rz @ Ry @ Rx
        X = (R[None] * elem[:, None, :]).sum(-1) + t
        Le, r = _nc(m.forward(p, X.detach()), y)
        hist.append(float((wt * Le).sum()))
        X.backward(m.adjoint(p, X.detach(), wt[:, None] * r, want_p0=False, want_x=True)[1])
        opt.step()
    return {"pose": torch.cat([a.detach(), t.detach()]), "losses": hist}


def _exact_tgv(u, w, alpha0=2.0, alpha1=1.0, eps=1e-3, scale=0.1):
    u, w = u.requires_grad_(True), w.requires_grad_(True)

    def fwd(x, a):
        d = torch.diff(x, dim=a)
        return torch.cat([d, torch.zeros_like(x.narrow(a, 0, 1))], dim=a)

    def bwd(x, a):
        d = torch.diff(x, dim=a)
        return torch.cat([torch.zeros_like(x.narrow(a, 0, 1)), d], dim=a)

    g2 = sum((fwd(u, a) - w[a]) ** 2 for a in range(3))
    e2 = sum((0.5 * (bwd(w[b], a) + bwd(w[a], b))) ** 2 for a in range(3) for b in range(3))
    val = scale * (alpha1 * (torch.sqrt(g2 + eps ** 2) - eps).sum() + alpha0 * (torch.sqrt(e2 + eps ** 2) - eps).sum())
    val.backward()
    return {"value": float(val.detach()), "grad_u": u.grad, "grad_w": w.grad}
