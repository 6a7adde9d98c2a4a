"""Cases that the framework's speed is measured on.

Each case is one call that a program makes through the public entry points: a forward
simulation, a checkpointed misfit gradient (plain or compressed, through ``DeviceShot``, the
autograd function or the 2-D batch call), or the codec on one wavefield.  The sizes are those
of the repository's own configurations (the two-layer, smooth-random, layered-noise and
fault-body models, the serving stream's three classes); 3-D runs take a few hundred of their
thousands of steps, with the source's band moved up so that the wave fills the model in them.

Inputs are seeded: a layered velocity with lateral variation, a Ricker source near the top
centre, receivers on a surface line or grid, and recorded traces with a few moveout events
(strong enough that the residual is as large as the data).  ``exact`` gives the same results
from the discrete equations in binary64 with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1810_05268_amd as P
from paper_1810_05268_amd.autograd import WaveProblem, wave_misfit
from paper_1810_05268_amd.shot import DeviceShot

VMAX = 3700.0     # upper bound of every velocity below: one time step and damping per grid


def _case(name, kind, n, order, nt, nbl=20, h=10.0, time_order=2, tol=0.0, slots=0.0, hint=0.0, shots=1,
          offgrid=False):
    """n: interior points per axis, x first (nz = 0: 2-D, whose second axis is depth).
    slots: checkpoint memory in uncompressed states (pairs of dense fields)."""
    n = tuple(n)
    return {"name": name, "kind": kind, "nx": n[0], "ny": n[1], "nz": n[2] if len(n) == 3 else 0, "nbl": nbl,
            "h": h, "order": order, "nt": nt, "time_order": time_order, "tol": tol, "slots": slots, "hint": hint,
            "shots": shots, "offgrid": offgrid}


def listed():
    return [
        # the small modelling call of a 2-D study: the two-layer model, launches and latency
        _case("forward2d_101", "forward", (101, 101), 4, 500),
        # one gradient of a 2-D inversion loop in torch (the smooth-random model), checkpoints compressed
        _case("autograd2d_400", "autograd", (400, 400), 8, 1000, h=5.0, tol=1e-4, slots=200),
        # the serving stream's 2-D class, alone, at its size and step count, with plain checkpoints
        _case("gradient2d_512", "gradient", (512, 512), 8, 1500, slots=60),
        # the same class under load: eight requests in one batch
        _case("batch2d_512", "batch", (512, 512), 8, 300, slots=30, shots=8),
        # 3-D modelling of the layered-noise model: data and final state
        _case("forward3d_128", "forward", (128, 128, 128), 8, 300),
        # the serving stream's medium 3-D class with plain checkpoints
        _case("gradient3d_160", "gradient", (160, 160, 160), 8, 200, slots=30),
        # a survey whose extents are no multiples of anything, receivers between grid points
        _case("gradient3d_ragged", "gradient", (141, 97, 83), 8, 200, nbl=21, slots=30, offgrid=True),
        # the serving stream's large class: order 12, compressed checkpoints, some recomputation
        _case("gradient3d_256", "gradient", (256, 256, 256), 12, 160, tol=1e-4, slots=6, hint=12.0),
        # the headline shot: order 16, 400^3 with its layers, every state compressed
        _case("gradient3d_320", "gradient", (320, 320, 320), 16, 100, nbl=40, h=12.5, tol=1e-4, slots=30),
        # fourth order in time
        _case("gradient3d_ot4", "gradient", (128, 128, 128), 8, 150, time_order=4, slots=40),
        # one large checkpoint through the codec, each way
        _case("encode3d_400", "encode", (400, 400, 400), 0, 0, nbl=0, tol=1e-4),
        _case("decode3d_400", "decode", (400, 400, 400), 0, 0, nbl=0, tol=1e-4),
    ]


def draw(rng):
    """One more case of the same ranges, no more work than the largest listed one."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["forward", "gradient", "gradient", "gradient", "autograd", "batch", "encode", "decode"])
    nd = 2 if kind == "batch" else rng.choice([2, 3, 3])
    if kind in ("encode", "decode"):
        n = [log(33, 1200) for _ in range(2)] if nd == 2 else [log(25, 400) for _ in range(3)]
        return _drawn(_case("", kind, n, 0, 0, nbl=0, tol=10.0 ** rng.uniform(-5.5, -2.5)))
    n = [log(41, 700) for _ in range(2)] if nd == 2 else [log(24, 300) for _ in range(3)]
    if rng.random() < 0.4:      # round sizes are as common as odd ones
        n = [max(16, 8 * round(v / 8)) for v in n]
    nt = log(60, 1000) if nd == 2 else log(40, 300)
    time_order = 4 if kind in ("forward", "gradient") and rng.random() < 0.15 else 2
    tol = 0.0 if rng.random() < 0.6 else 10.0 ** rng.uniform(-5.0, -3.0)
    # compressed autograd calls plan later calls from the first, so they get memory for all states
    slots = nt / 2.0 + 2 if kind == "autograd" else rng.uniform(3.0, max(4.0, nt / 4.0))
    c = _case("", kind, n, rng.choice([4, 8, 8, 12, 16]), nt, nbl=rng.choice([10, 20, 20, 31, 40]),
              h=rng.choice([5.0, 10.0, 12.5]), time_order=time_order, tol=tol, slots=slots,
              hint=4.0 if tol > 0 and kind != "autograd" else 0.0,
              shots=rng.randint(2, 8) if kind == "batch" else 1, offgrid=rng.random() < 0.3)
    most = max(work(x)["bytes"] for x in listed())
    while work(c)["bytes"] > 0.7 * most and c["nt"] > 20:   # recomputation comes on top
        c["nt"] = c["nt"] * 3 // 4
    # memory stays a few GB and a run needs no more slots than steps
    c["slots"] = min(c["slots"], 12e9 / (8.0 * _points(c)), c["nt"] + 2.0)
    return _drawn(c)


def _drawn(c):
    del c["name"]
    return c


# ---------------------------------------------------------------- geometry and inputs

def _n(c):
    return (c["nx"], c["ny"], c["nz"]) if c["nz"] else (c["nx"], c["ny"])


def _points(c):
    return math.prod(v + 2 * c["nbl"] for v in _n(c))


def _dt(c):
    nd = len(_n(c))
    a = _fd_weights(c["order"] // 2)
    s = abs(a[0]) + 2 * sum(abs(v) for v in a[1:])
    lim = 2.0 if c["time_order"] == 2 else math.sqrt(12.0)
    return 0.4 * lim / (VMAX * math.sqrt(nd * s / c["h"] ** 2))


def _fd_weights(k_max):
    f = math.factorial
    a = [0.0] + [2.0 * (-1) ** (k + 1) * f(k_max) ** 2 / (k * k * f(k_max - k) * f(k_max + k))
                 for k in range(1, k_max + 1)]
    a[0] = -2.0 * sum(a)
    return a


class _Inputs:
    """Host arrays of one shot, from the case and the seed alone."""

    def __init__(self, c, seed):
        rng = np.random.default_rng(seed)
        n, h, nbl = _n(c), c["h"], c["nbl"]
        self.nd, self.dt = len(n), _dt(c)
        nz = n[-1]
        layers = int(rng.integers(3, 8))
        speed = np.sort(rng.uniform(1500.0, 3400.0, size=layers))
        prof = speed[np.minimum(np.arange(nz) * layers // nz, layers - 1)]
        shape = tuple(reversed(n))
        wave = np.zeros((1,) * self.nd)
        for ax in range(self.nd):
            m = shape[ax]
            view = [1] * self.nd
            view[ax] = m
            wave = wave + np.sin(2 * np.pi * (rng.uniform(1, 5) * np.arange(m) / m + rng.uniform())).reshape(view)
        self.vel = np.ascontiguousarray(prof.reshape((nz,) + (1,) * (self.nd - 1)) * (1 + 0.02 * wave),
                                        dtype=np.float32)
        depth = 2 * h
        self.src = np.array([[(m - 1) * h / 2.0 for m in n[:-1]] + [depth]])
        off = 0.3 * h if c["offgrid"] else 0.0
        line = [np.minimum(np.arange(m) * h + off, (m - 1) * h) for m in n[:-1]]
        grid = np.meshgrid(*reversed(line), indexing="ij")
        self.rec = np.stack([g.ravel() for g in reversed(grid)] + [np.full(grid[0].size, depth + off)], axis=1)
        # the source's band: its onset lies within the first fifth of the run
        f0 = rng.uniform(0.8, 1.2) * max(10.0, 6.0 / (c["nt"] * self.dt))
        t = np.arange(c["nt"]) * self.dt - 1.0 / f0
        self.wavelet = _ricker(t, f0).astype(np.float32)
        self.f0, self.events = f0, rng.uniform(size=(4, 3))

    def d_obs(self, c, device):
        """Recorded traces: direct wave and reflections with moveout, binary32 [nt+1][nrec]."""
        t = torch.arange(c["nt"] + 1, dtype=torch.float64, device=device)[:, None] * self.dt
        end = c["nt"] * self.dt
        x = torch.as_tensor(np.linalg.norm(self.rec - self.src, axis=1), device=device)[None, :]
        out = torch.zeros((c["nt"] + 1, x.shape[1]), dtype=torch.float32, device=device)
        for a, b, v in self.events:
            arrive = 1.0 / self.f0 + torch.sqrt((0.7 * end * b) ** 2 + (x / (1500.0 + 1500.0 * v)) ** 2)
            out += ((a - 0.5) * c["h"] / (x + 5 * c["h"]) * _ricker(t - arrive, self.f0)).to(torch.float32)
        return out


def _ricker(t, f0):
    a = (math.pi * f0 * t) ** 2
    return (1.0 - 2.0 * a) * (torch.exp(-a) if isinstance(a, torch.Tensor) else np.exp(-a))


def _field(c, seed, device):
    """A wavefield part way through a run: wavefronts around a source near the top, zero ahead of them."""
    rng = np.random.default_rng(seed)
    shape = tuple(reversed(_n(c)))
    m = max(shape)
    ax = [torch.arange(s, dtype=torch.float64, device=device).reshape([-1 if i == a else 1 for i in range(len(shape))])
          for a, s in enumerate(shape)]
    out = torch.zeros(shape, dtype=torch.float32, device=device)
    for _ in range(5):
        centre = [rng.uniform(-0.3, 0.4) * shape[0]] + [s * rng.uniform(0.3, 0.7) for s in shape[1:]]
        r = torch.sqrt(sum((x - x0) ** 2 for x, x0 in zip(ax, centre)))
        out += (rng.uniform(2.0, 8.0) / (r + 10.0) *
                _ricker(r - rng.uniform(0.2, 0.6) * m, rng.uniform(0.02, 0.05))).to(torch.float32)
    return out


# ---------------------------------------------------------------- the calls

def _pad(v, nbl):
    return np.ascontiguousarray(np.pad(v, nbl, mode="edge"))


def _shot(c, inp):
    n, nd = _n(c), inp.nd
    return DeviceShot(nd, n, (c["h"],) * nd, c["nbl"], c["order"], c["nt"], inp.dt, VMAX, _pad(inp.vel, c["nbl"]),
                      inp.wavelet, inp.src, inp.rec, time_order=c["time_order"])


def _budget(c):
    return int(c["slots"] * 8 * _points(c))


def prepare(case, seed):
    c, dev = case, "cuda"
    if c["kind"] in ("encode", "decode"):
        f = _field(c, seed, dev)
        dims = list(_n(c))
        nd = len(dims)
        # a checkpoint's stream takes far less than the worst case; a caller sizes it by half the raw field
        out = torch.zeros(min(P.zfpk_max_bytes(nd, dims), 2 * f.numel() + (1 << 16)), dtype=torch.uint8, device=dev)
        ws = torch.empty(P.zfpk_workspace_bytes(nd, dims), dtype=torch.uint8, device=dev)
        st = {"c": c, "field": f, "stream": out, "ws": ws}
        if c["kind"] == "decode":
            st["nbytes"] = P.zfpk_encode(f, c["tol"], out, ws)
            st["field"] = torch.empty_like(f)
        return st
    if c["kind"] == "autograd":
        i = _Inputs(c, seed)
        problem = WaveProblem(i.nd, _n(c), (c["h"],) * i.nd, c["nbl"], c["order"], c["nt"], i.dt, VMAX, i.wavelet,
                              i.src, i.rec, i.d_obs(c, dev), _budget(c), tol=c["tol"])
        return {"c": c, "problem": problem, "vel": torch.as_tensor(i.vel, device=dev).requires_grad_(True)}
    inps = [_Inputs(c, seed * 1000 + k) for k in range(c["shots"])]
    shots = [_shot(c, i) for i in inps]
    if c["kind"] == "forward":
        return {"c": c, "shot": shots[0]}
    d_obs = [i.d_obs(c, dev) for i in inps]
    if c["kind"] == "gradient":
        return {"c": c, "shot": shots[0], "d_obs": d_obs[0]}
    pbs = [s.pb for s in shots]
    ws = torch.empty(P.batch_workspace_bytes(pbs, _budget(c)) + 256, dtype=torch.uint8, device=dev)
    ws = ws[(-ws.data_ptr()) % 256:]
    grads = [torch.empty(s.shape, dtype=torch.float64, device=dev) for s in shots]
    return {"c": c, "shots": shots, "d_obs": d_obs, "ws": ws, "grads": grads}


def run(state):
    s, c = state, state["c"]
    if c["kind"] == "encode":
        nbytes = P.zfpk_encode(s["field"], c["tol"], s["stream"], s["ws"])
        return {"nbytes": nbytes, "stream": s["stream"]}   # zeros after the stream
    if c["kind"] == "decode":
        P.zfpk_decode(s["stream"], s["field"], s["nbytes"])
        return {"field": s["field"]}
    if c["kind"] == "autograd":
        s["vel"].grad = None
        phi = wave_misfit(s["vel"], s["problem"])
        phi.backward()
        return {"phi": phi.detach(), "grad": s["vel"].grad}
    if c["kind"] == "forward":
        data, u = s["shot"].forward(want_state=True)
        return {"data": data, "state": u}
    if c["kind"] == "gradient":
        phi, g, _, d_sim = s["shot"].misfit_gradient(s["d_obs"], _budget(c), c["tol"], c["hint"], want_dsim=True)
        return {"phi": phi, "grad": g, "d_sim": d_sim}
    phis, _ = P.batch_misfit_gradient([x.pb for x in s["shots"]], s["d_obs"], _budget(c), c["tol"], s["grads"],
                                      s["ws"], ratio_hint=c["hint"])
    return {"phi": phis, "grad": s["grads"]}


def work(case):
    """A forward step reads u^n, u^{n-1} and w and writes u^{n+1}; an adjoint step reads u^k and updates the
    binary64 gradient besides; fourth order in time takes two passes.  Recomputation is not counted."""
    c, p = case, _points(case)
    if c["kind"] in ("encode", "decode"):
        return {"bytes": 4.2 * p, "flops": 30.0 * p}
    nd, k = len(_n(c)), c["order"] // 2
    lap = nd * (3 * k + 1)
    fwd, adj, pt = (16, 36, lap + 8) if c["time_order"] == 2 else (32, 68, 2 * lap + 12)
    steps = float(p) * c["nt"] * c["shots"]
    if c["kind"] == "forward":
        return {"bytes": fwd * steps, "flops": pt * steps}
    return {"bytes": (fwd + adj) * steps, "flops": (2 * pt + 4) * steps}


# ---------------------------------------------------------------- the same in binary64

class _Discrete:
    """The discrete equations in binary64 torch: leapfrog on a padded grid with zero halo."""

    def __init__(self, c, inp, device):
        self.c, self.dev = c, device
        self.k = c["order"] // 2
        vel = torch.as_tensor(_pad(inp.vel, c["nbl"]), device=device).double()
        self.vel, self.w = vel, inp.dt ** 2 * vel * vel
        self.shape, self.dt = vel.shape, inp.dt
        self.a = torch.zeros((1,) * inp.nd, dtype=torch.float64, device=device)
        if c["nbl"]:
            smax = 3 * VMAX * math.log(1000.0) / (2 * c["nbl"] * c["h"])
            for ax, m in enumerate(self.shape):
                i = torch.arange(m, dtype=torch.float64, device=device)
                d = torch.clamp(torch.maximum(c["nbl"] - i, i - (m - 1 - c["nbl"])), min=0.0)
                view = [-1 if q == ax else 1 for q in range(inp.nd)]
                self.a = self.a + (0.5 * inp.dt * smax * (d / c["nbl"]) ** 2).reshape(view)
        self.a = self.a.expand(self.shape).contiguous()
        self.wt = _fd_weights(self.k)
        self.src, self.rec = self.points(inp.src), self.points(inp.rec)
        self.q = inp.wavelet.astype(np.float64)

    def points(self, xyz):
        """Flat indices and multilinear weights [npoints][2^d]."""
        nd = xyz.shape[1]
        g = xyz / self.c["h"] + self.c["nbl"]
        ext = list(reversed(self.shape))
        i0 = np.minimum(np.floor(g).astype(np.int64), np.array(ext) - 2)
        fr = g - i0
        idx, wt = [], []
        for corner in range(2 ** nd):
            p, w, stride = 0, 1.0, 1
            for d in range(nd):
                b = (corner >> d) & 1
                p = p + (i0[:, d] + b) * stride
                stride *= ext[d]
                w = w * (fr[:, d] if b else 1.0 - fr[:, d])
            idx.append(p)
            wt.append(w)
        return (torch.as_tensor(np.stack(idx, 1), device=self.dev), torch.as_tensor(np.stack(wt, 1), device=self.dev))

    def lap(self, u):
        out = (u.dim() * self.wt[0]) * u
        for ax in range(u.dim()):
            m = u.shape[ax]
            for k in range(1, min(self.k, m - 1) + 1):
                out.narrow(ax, 0, m - k).add_(u.narrow(ax, k, m - k), alpha=self.wt[k])
                out.narrow(ax, k, m - k).add_(u.narrow(ax, 0, m - k), alpha=self.wt[k])
        return out / self.c["h"] ** 2

    def term(self, u, points, vals):
        """w (B u + injected vals), and w lap u."""
        v = self.w * self.lap(u)
        t = v + self.w / 12.0 * self.lap(v) if self.c["time_order"] == 4 else v.clone()
        s = torch.zeros(u.numel(), dtype=torch.float64, device=self.dev)
        s.index_add_(0, points[0].reshape(-1), (points[1] * vals).reshape(-1))
        return t + self.w * s.view_as(u), v

    def advance(self, u, prev, t):
        return (2 * u - (1 - self.a) * prev + t) / (1 + self.a)

    def sample(self, u):
        return (u.reshape(-1)[self.rec[0]] * self.rec[1]).sum(1)

    def forward(self, keep):
        u = torch.zeros(self.shape, dtype=torch.float64, device=self.dev)
        prev, traj, rows = u, [u], [self.sample(u)]
        for n in range(self.c["nt"]):
            t, _ = self.term(u, self.src, float(self.q[n]))
            u, prev = self.advance(u, prev, t), u
            rows.append(self.sample(u))
            if keep:
                traj.append(u)
        return torch.stack(rows), traj if keep else torch.stack([u, prev])

    def gradient(self, d_obs):
        d_sim, traj = self.forward(True)
        res = d_sim - d_obs.double()
        res[0] = 0.0
        lam = torch.zeros(self.shape, dtype=torch.float64, device=self.dev)
        nxt, g = lam, torch.zeros_like(lam)
        for k in range(self.c["nt"], 0, -1):
            t, v = self.term(lam, self.rec, res[k][:, None])
            u = traj.pop()
            g += u * t
            if self.c["time_order"] == 4:
                g += v * (self.w * self.lap(u)) / 12.0
            lam, nxt = self.advance(lam, nxt, t), lam
        return 0.5 * float((res ** 2).sum()), g * (-1.0 / self.dt ** 2), d_sim

    def interior_gradient(self, g):
        """d phi / d c on the interior: dm/dc = -2/c^3 and the adjoint of the edge padding."""
        g, b = g * (-2.0 / self.vel ** 3), self.c["nbl"]
        for ax, m in enumerate(self.shape):
            out = g.narrow(ax, b, m - 2 * b).clone()
            if b:
                out.narrow(ax, 0, 1).add_(g.narrow(ax, 0, b).sum(ax, keepdim=True))
                out.narrow(ax, m - 2 * b - 1, 1).add_(g.narrow(ax, m - b, b).sum(ax, keepdim=True))
            g = out
        return g


def exact(case, seed):
    c = case
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if c["kind"] == "encode":
        return None       # bytes
    if c["kind"] == "decode":
        return {"field": _field(c, seed, dev).double()}
    if c["kind"] == "autograd":
        inp = _Inputs(c, seed)
        d = _Discrete(c, inp, dev)
        phi, g, _ = d.gradient(inp.d_obs(c, dev))
        return {"phi": torch.tensor(phi, dtype=torch.float64), "grad": d.interior_gradient(g)}
    inps = [_Inputs(c, seed * 1000 + k) for k in range(c["shots"])]
    if c["kind"] == "forward":
        data, state = _Discrete(c, inps[0], dev).forward(False)
        return {"data": data, "state": state}
    got = [_Discrete(c, i, dev).gradient(i.d_obs(c, dev)) for i in inps]
    if c["kind"] == "gradient":
        return {"phi": got[0][0], "grad": got[0][1], "d_sim": got[0][2]}
    return {"phi": [g[0] for g in got], "grad": [g[1] for g in got]}
