"""The work a program has this package do, as cases that can be timed.

A case is a dict of plain values; `kind` names the path it takes:

* gradient   one gradient iteration on a D2Q9 lattice: forward solve, cost and
             adjoint seed, AMRT sweep, gradient and norms, control update
             (`GradientIteration.step`), or with `op` = "lma" the gradient and
             the linearised line minimisation's step size for it, from one
             tangent solve (`lma_zeta`), the control left as it is;
* forward    one forward solve without an adjoint record and its cost, what a
             line search asks for at every trial control;
* autograd   `MRTSolve` inside a torch program: forward, loss, backward, with
             the trajectory recomputed from checkpoints;
* d3q19      one gradient iteration on a three-dimensional lattice;
* batch      one gradient iteration of many uneven periodic problems together;
* score      the surrogate network on a batch of candidate controls;
* train      training steps of the surrogate on random crops.

Inputs are drawn from the seed alone, with the distributions of the package's
own workloads: u0 = 1 +- 10 % noise, control and target bumps, symmetric
positive definite tensors, disk (sphere) masks inside a solid ring (frame).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1908_03876_amd import abi
from paper_1908_03876_amd.autograd import MRTSolve
from paper_1908_03876_amd.batched import Batch
from paper_1908_03876_amd.inputs import Problem, Problem3
from paper_1908_03876_amd.solver import DeviceProblem, GradientIteration, Tape
from paper_1908_03876_amd.solver3 import DeviceProblem3, GradientIteration3
from paper_1908_03876_amd.surrogate import SHAPES, Surrogate

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "f64": torch.float64}


def listed():
    g = dict(kind="gradient", op="step", dtype="f32", mask=True, source=1, species=2, ckpt=0)
    return [
        # the plain method in double precision on a small periodic lattice:
        # hundreds of dependent steps of a few microseconds each
        dict(g, name="gradient 64 f64", nx=64, ny=64, steps=200, dtype="f64", mask=False),
        # the small copy of the masked workload, a first experiment's size
        dict(g, name="gradient 128 masked", nx=128, ny=128, steps=200),
        # one trial of a line search on an odd-shaped domain
        dict(kind="forward", name="forward 301x157", nx=301, ny=157, steps=300, dtype="f32",
             mask=True, source=1, species=2),
        # a gradient with its linearised line minimisation, on a middling
        # lattice that the caches hold
        dict(g, name="lma 512 masked", nx=512, ny=512, steps=100, op="lma"),
        # differentiation form: checkpoints and recomputation under autograd
        dict(kind="autograd", name="autograd 1024", nx=1024, ny=1024, steps=200, ckpt=50,
             dtype="f32", mask=True),
        # the default workload's lattice at a shorter horizon
        dict(g, name="gradient 2048 masked", nx=2048, ny=2048, steps=100),
        # the implicit second-order source on a ragged periodic box
        dict(g, name="implicit 900x700", nx=900, ny=700, steps=80, mask=False, source=3),
        # attraction and repulsion: the third species
        dict(g, name="three species 1024", nx=1024, ny=1024, steps=60, species=3),
        # the three-dimensional porous workload
        dict(kind="d3q19", name="d3q19 256 porous", nx=256, ny=256, nz=256, steps=16,
             dtype="f32", mask=True, ckpt=0),
        # many uneven problems at once, checkpointed and replayed as a graph
        dict(kind="batch", name="batch of 16", count=16, steps=100, ckpt=25, dtype="f32",
             sizes="128,256,384,512,768,1024"),
        # candidate steps scored by the surrogate
        dict(kind="score", name="score 17x1024", batch=17, h=1024, w=1024),
        # surrogate training
        dict(kind="train", name="train 64x64", batch=64, crop=64, steps=4, pool=64, size=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gradient", "gradient", "gradient", "forward", "lma", "autograd",
                       "d3q19", "batch", "score", "train"])
    if kind in ("gradient", "forward", "lma", "autograd"):
        nx, ny = _log(rng, 40, 2048), _log(rng, 40, 2048)
        steps = min(_log(rng, 30, 300), max(8, int(1.0e8 / (nx * ny))))
        mask, dtype = rng.random() < 0.6, "f64" if rng.random() < 0.25 else "f32"
        c = dict(kind=kind, nx=nx, ny=ny, steps=steps, dtype=dtype, mask=mask)
        if kind == "autograd":
            c["ckpt"] = max(2, steps // rng.randint(2, 6))
            return c
        c["source"], c["species"] = rng.choice([(1, 2), (1, 2), (1, 2), (3, 2), (1, 3)])
        if kind != "forward":
            c["ckpt"] = 0 if rng.random() < 0.7 else max(2, steps // rng.randint(2, 5))
            c["op"] = "lma" if kind == "lma" else "step"
            c["kind"] = "gradient"
        return c
    if kind == "d3q19":
        n = [_log(rng, 16, 160) for _ in range(3)]
        steps = min(_log(rng, 6, 40), max(4, int(5.0e7 / (n[0] * n[1] * n[2]))))
        return dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], steps=steps, ckpt=0,
                    dtype="f64" if rng.random() < 0.2 else "f32", mask=rng.random() < 0.6)
    if kind == "batch":
        sizes = sorted(_log(rng, 64, 700) for _ in range(4))
        steps = _log(rng, 30, 100)
        return dict(kind=kind, count=rng.randint(3, 16), steps=steps, ckpt=max(2, steps // 4),
                    dtype="f64" if rng.random() < 0.2 else "f32",
                    sizes=",".join(str(s) for s in sizes))
    if kind == "score":
        h, w = _log(rng, 64, 1024), _log(rng, 64, 1024)
        return dict(kind=kind, batch=rng.randint(1, 17), h=h, w=w)
    return dict(kind="train", batch=_log(rng, 8, 64), crop=rng.randint(24, 64),
                steps=rng.randint(2, 4), pool=64, size=rng.randint(96, 256))


# ------------------------------------------------------------------- inputs

def _spd(rng, dim):
    d = rng.uniform(0.1, 1.0, dim)
    r = np.eye(dim)
    for a in range(dim):
        for b in range(a):
            r[a, b] = r[b, a] = rng.uniform(-0.3, 0.3)
    return r * np.sqrt(np.outer(d, d))


def _bumps(shape, rng, count, sigma, amps, periodic):
    """Sum of Gaussian bumps, an outer product of one profile per axis."""
    out = np.zeros(shape)
    for k in range(count):
        term = np.full((1,) * len(shape), float(amps[k]))
        for axis, n in enumerate(shape):
            d = np.abs(np.arange(n) - rng.uniform(0, n))
            d = np.minimum(d, n - d) if periodic else d
            view = [1] * len(shape)
            view[axis] = n
            term = term * np.exp(-d * d / (2.0 * sigma * sigma)).reshape(view)
        out += term
    return out


def _mask(shape, rng, count, rmin, rmax):
    """Solid disks (spheres) inside a one-cell solid ring (frame)."""
    solid = np.zeros(shape, dtype=np.uint8)
    for _ in range(count):
        c = [rng.uniform(0, n) for n in shape]
        r = int(rng.integers(rmin, rmax + 1))
        box = [slice(max(0, int(x - r)), min(n, int(x + r) + 2)) for x, n in zip(c, shape)]
        d2 = sum((g - x) ** 2 for g, x in zip(np.ogrid[tuple(box)], c))
        solid[tuple(box)] |= (d2 <= r * r).astype(np.uint8)
    for axis in range(len(shape)):
        for end in (0, -1):
            at = [slice(None)] * len(shape)
            at[axis] = end
            solid[tuple(at)] = 1
    return solid


def _fields(case, seed):
    """Everything one problem is made of, as a dict of arrays and numbers."""
    rng = np.random.default_rng([int(seed), case["nx"], case["ny"]])
    shape = (case["ny"], case["nx"]) if "nz" not in case else (case["nz"], case["ny"], case["nx"])
    dim, n = len(shape), min(shape)
    solid = None
    if case["mask"]:
        if dim == 2:
            count = max(4, int(200 * shape[0] * shape[1] / 2048 ** 2))
            solid = _mask(shape, rng, count, min(5, n // 16), min(30, max(3, n // 16)))
        else:
            solid = _mask(shape, rng, max(3, shape[0] * shape[1] * shape[2] // 16000),
                          max(2, n // 64), max(2, n // 24))
    p = dict(Du=_spd(rng, dim), Dv=_spd(rng, dim), Cchi=_spd(rng, dim), chi=0.5, solid=solid,
             periodic=solid is None, alpha=1e-3)
    p["u0"] = 1.0 + 0.1 * rng.uniform(-1, 1, shape)
    p["v0"] = np.zeros(shape)
    sigma = max(max(shape) / 8.0, 4.0)
    p["control"] = _bumps(shape, rng, 2, sigma, rng.uniform(-5, 5, 2), p["periodic"])
    p["u_target"] = 1.0 + _bumps(shape, rng, 4, sigma, [0.5] * 4, p["periodic"])
    if case.get("species", 2) == 3:
        p.update(Dw=_spd(rng, dim), Cw=_spd(rng, dim), chi_w=-0.4, a_w=0.5, b_w=0.8, s_w=0.05,
                 sw=rng.uniform(0.8, 1.6, 7), w0=0.2 * rng.uniform(0, 1, shape))
    if solid is not None:
        for name in ("u0", "control", "u_target", "w0"):
            if name in p:
                p[name][solid != 0] = 0.0
    return p


def _problem(case, seed):
    p = _fields(case, seed)
    if "nz" in case:
        return Problem3(nx=case["nx"], ny=case["ny"], nz=case["nz"], nsteps=case["steps"], **p)
    extra = dict(nspecies=3) if case.get("species", 2) == 3 else {}
    return Problem(nx=case["nx"], ny=case["ny"], nsteps=case["steps"],
                   source_term=case.get("source", 1), **extra, **p)


def _batch_cases(case):
    sizes = [int(s) for s in case["sizes"].split(",")]
    picks = [sizes[k % len(sizes)] for k in range(case["count"])]
    np.random.default_rng(case["count"]).shuffle(picks)
    return [dict(nx=L, ny=L, steps=case["steps"], mask=False) for L in picks]


def _network(seed):
    """Weights that bfloat16 holds exactly, as (weight, bias) per layer."""
    rng = np.random.default_rng([int(seed), 10])
    out = []
    for o, c in SHAPES:
        w = rng.normal(0.0, 1.0 / math.sqrt(9 * c), (o, c, 3, 3))
        b = rng.normal(0.0, 0.05, o)
        out.append(tuple(torch.tensor(a, dtype=torch.float32).bfloat16().double().numpy()
                         for a in (w, b)))
    return out


def _images(seed, n, h, w):
    """n smooth controls of a few units, [n, h, w] on the device."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 7 + 1)
    ay = torch.arange(h, device=DEV, dtype=torch.float32)
    ax = torch.arange(w, device=DEV, dtype=torch.float32)
    out = torch.zeros((n, h, w), device=DEV)
    for _ in range(4):
        r = torch.rand((4, n, 1), generator=gen, device=DEV)
        s = 4.0 + 28.0 * r[2]
        gy = torch.exp(-((ay[None] - h * r[0]) / s) ** 2 / 2) * (10.0 * r[3] - 5.0)
        gx = torch.exp(-((ax[None] - w * r[1]) / s) ** 2 / 2)
        out += gy[:, :, None] * gx[:, None, :]
    return out


# ------------------------------------------------------------ prepare and run

def prepare(case, seed):
    k, dt = case["kind"], DTYPES[case.get("dtype", "f32")]
    if k == "gradient":
        dp = DeviceProblem(_problem(case, seed), dtype=dt, device=DEV)
        return dict(case=case, it=GradientIteration(dp, ckpt_every=case["ckpt"] or -1))
    if k == "forward":
        dp = DeviceProblem(_problem(case, seed), dtype=dt, device=DEV)
        return dict(case=case, dp=dp, tape=Tape(dp, 0), uN=dp.empty_field(), vN=dp.empty_field())
    if k == "autograd":
        p = _problem(case, seed)
        s = MRTSolve(p, dtype=dt, device=DEV, ckpt_every=case["ckpt"])
        on = lambda a: torch.tensor(a, dtype=dt, device=DEV)  # noqa: E731
        return dict(case=case, solve=s, c=on(p.control).requires_grad_(True), target=on(p.u_target),
                    fluid=on(p.fluid.astype(float)))
    if k == "d3q19":
        dp = DeviceProblem3(_problem(case, seed), dtype=dt, device=DEV)
        return dict(case=case, it=GradientIteration3(dp, ckpt_every=case["ckpt"] or -1))
    if k == "batch":
        ps = [_problem(c, seed * 100 + i) for i, c in enumerate(_batch_cases(case))]
        return dict(case=case, batch=Batch(ps, dtype=dt, ckpt_every=case["ckpt"], device=DEV))
    if k == "score":
        s = Surrogate(case["batch"], case["h"], case["w"], device=DEV)
        s.load(_network(seed))
        return dict(case=case, net=s, x=_images(seed, case["batch"], case["h"], case["w"]))
    s = Surrogate(case["batch"], case["crop"], case["crop"], device=DEV)
    s.load(_network(seed))
    x = _images(seed, case["pool"], case["size"], case["size"])
    y = 0.02 * _images(seed + 1, case["pool"], case["size"], case["size"])
    grads = [torch.empty(abi.mrt_srg_param(s.handle, layer, kind)[1], device=DEV)
             for layer in range(4) for kind in range(4)]
    return dict(case=case, net=s, x=x, y=y, grads=grads, seed=int(seed) % 65536)


def run(st):
    case = st["case"]
    k = case["kind"]
    if k == "gradient":
        it = st["it"]
        r = it.gradient() if case["op"] == "lma" else it.step()
        zeta = it.lma_zeta() if case["op"] == "lma" else r["zeta"]
        nx = it.dp.nx
        out = dict(grad=it.grad[:, :nx], uN=it.uN[:, :nx], vN=it.vN[:, :nx],
                   scalars=np.float32([r["J"], zeta]))
        moved = it.duN if case["op"] == "lma" else it.dp.control
        out["tangent" if case["op"] == "lma" else "control"] = moved[:, :nx]
        return out
    if k == "forward":
        dp = st["dp"]
        abi.mrt_forward(dp.struct, st["tape"].handle, dp.u0, dp.v0, dp.control, None, st["uN"],
                        st["vN"])
        r = abi.cost_gradient(dp.struct, st["tape"].handle, st["uN"], dp.u_target, dp.control)
        return dict(uN=st["uN"][:, :dp.nx], vN=st["vN"][:, :dp.nx], J=np.float32(r["J"]))
    if k == "autograd":
        c = st["c"]
        c.grad = None
        uN, vN = st["solve"](c)
        loss = 0.5 * (((uN - st["target"]) * st["fluid"]) ** 2).sum() + 0.5e-3 * (c * c).sum()
        loss.backward()
        return dict(grad=c.grad, uN=uN.detach(), vN=vN.detach())
    if k == "d3q19":
        it = st["it"]
        r = it.step()
        nx = it.dp.nx
        return dict(grad=it.grad[..., :nx], uN=it.uN[..., :nx], vN=it.vN[..., :nx],
                    control=it.dp.control[..., :nx], scalars=np.float32([r["J"], r["zeta"]]))
    if k == "batch":
        b = st["batch"]
        b.iterate(use_graph=True)
        got = b.scalars()
        return dict(J=np.float32([s["J"] for s in got]),
                    each=[[b.get(i, name) for name in ("grad", "uN", "control")]
                          for i in range(b.count)])
    if k == "score":
        return st["net"].forward(st["x"])
    s = st["net"]
    loss = s.train(st["x"], st["y"], steps=case["steps"], batch=case["batch"], crop=case["crop"],
                   seed=st["seed"], log_every=1000)
    for i, t in enumerate(st["grads"]):
        abi.mrt_srg_copy_param(s.handle, i // 4, i % 4, False, t)
    return dict(params=st["grads"], loss=np.float32(loss))


# ----------------------------------------------------------------------- work

# arithmetic of one node and step, counted on the scheme: moments, relaxation
# of every species, sources (the adjoint also sums weighted populations)
_FLOPS = {("d2q9", 2): (270, 320, 320), ("d2q9", 3): (410, 480, 480), ("d3q19", 2): (700, 760, 760)}


def work(case):
    """Bytes: the fields that come in and go out once and, where a gradient is
    taken, the trajectory's record (u and the first moments), written and
    read once.  Operations: every step of every sweep once."""
    k = case["kind"]
    if k in ("score", "train"):
        per = 2 * 9 * (32 + 32 * 32 + 32 * 32 + 32)
        if k == "score":
            n = case["batch"] * case["h"] * case["w"]
            return dict(bytes=8.0 * n, flops=float(per * n))
        n = case["batch"] * case["crop"] ** 2 * case["steps"]
        return dict(bytes=16.0 * n, flops=3.0 * per * n)
    el = 8 if case["dtype"] == "f64" else 4
    if k == "batch":
        cells = sum(c["nx"] ** 2 for c in _batch_cases(case))
    else:
        cells = case["nx"] * case["ny"] * case.get("nz", 1)
    sp = case.get("species", 2)
    fwd, adj, tan = _FLOPS[("d3q19" if k == "d3q19" else "d2q9", sp)]
    steps = float(case["steps"]) * cells
    if k == "forward":
        return dict(bytes=6.0 * el * cells, flops=fwd * steps)
    rec = {("d2q9", 2): 3, ("d2q9", 3): 5, ("d3q19", 2): 4}[("d3q19" if k == "d3q19" else "d2q9", sp)]
    lma = case.get("op") == "lma"
    return dict(bytes=8.0 * el * cells + (3 if lma else 2) * rec * el * steps,
                flops=(fwd + adj + (tan if lma else 0)) * steps)


# ---------------------------------------------------------------------- exact

class _Exact:
    """The scheme in float64 with dense matrices: collide, then stream with
    halfway bounce-back; gradients by reverse-mode steps."""

    def __init__(self, p, steps, source=1):
        on = lambda a: torch.tensor(np.asarray(a, dtype=np.float64), device=DEV)  # noqa: E731
        self.steps, self.source, self.p = steps, source, p
        self.shape = p["u0"].shape
        dim = len(self.shape)
        if dim == 2:
            e = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
            w = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
        else:
            e = [(a, b, c) for c in (-1, 0, 1) for b in (-1, 0, 1) for a in (-1, 0, 1)
                 if abs(a) + abs(b) + abs(c) <= 2]
            w = [{0: 1 / 3, 1: 1 / 18, 2: 1 / 36}[sum(map(abs, x))] for x in e]
        self.e, E, W = e, np.array(e, dtype=float), np.array(w)
        self.w, self.E = on(W), on(E)
        self.opp = [e.index(tuple(-x for x in v)) for v in e]
        self.solid = None if p["solid"] is None else torch.tensor(p["solid"] != 0, device=DEV)
        if self.solid is not None:
            self.wall = [self._roll(self.solid, i) for i in range(len(e))]
        names = ["u", "v"] + (["w"] if "Dw" in p else [])
        K = {s: np.linalg.inv(p["D" + s] * 3.0 + 0.5 * np.eye(dim)) for s in names}
        self.A = [on(self._relaxation(K[s], E, W, p.get("s" + s))) for s in names]
        B = lambda chi, C, s: on(-3.0 * chi * K["u"] @ C @ K[s])  # noqa: E731
        self.B = [B(p["chi"], p["Cchi"], "v")] + ([B(p["chi_w"], p["Cw"], "w")] if "Dw" in p else [])
        first = ["u0", "v0", "w0"][: len(names)]
        t0 = torch.stack([on(p[n]) for n in first]).reshape(len(names), 1, -1)
        self.f0 = self.w[None, :, None] * t0
        self.c = on(p["control"]).reshape(-1)
        self.target = on(p["u_target"]).reshape(-1)
        self.fluid = on(np.ones(self.shape) if p["solid"] is None else p["solid"] == 0).reshape(-1)

    @staticmethod
    def _relaxation(K, E, W, rates):
        """I - M^-1 Pi (M - m_eq 1^T): post-collision populations, linearly."""
        q, dim = E.shape
        if dim == 2:
            e2 = (E * E).sum(1)
            x, y = E[:, 0], E[:, 1]
            M = np.stack([np.ones(q), 3 * e2 - 4, 4.5 * e2 * e2 - 10.5 * e2 + 4, x,
                          (3 * e2 - 5) * x, y, (3 * e2 - 5) * y, x * x - y * y, x * y])
            s = np.ones(7) if rates is None else rates
            Pi = np.diag([s[0], s[1], s[2], 0, s[3], 0, s[4], s[5], s[6]])
            Pi[np.ix_([3, 5], [3, 5])] = K
            C = np.linalg.solve(M, Pi @ M)
        else:  # unit rates: only the flux rows relax differently
            n = (E[:, 0] ** 2).sum()
            C = np.eye(q) + E @ (K - np.eye(dim)) @ E.T / n
        return np.eye(q) - C + np.outer(C @ W, np.ones(q))

    def _roll(self, a, i):
        axes = list(range(a.dim() - len(self.shape), a.dim()))
        return torch.roll(a, tuple(reversed(self.e[i])), axes)  # a(x - e_i)

    def _stream(self, f):
        g = f.reshape(f.shape[0], f.shape[1], *self.shape)
        out = []
        for i in range(len(self.e)):
            a = self._roll(g[:, i], i)
            if self.solid is not None:
                a = torch.where(self.wall[i], g[:, self.opp[i]], a)
                a = torch.where(self.solid, torch.zeros_like(a), a)
            out.append(a)
        return torch.stack(out, 1).reshape(f.shape)

    def _kinetics(self, s, c):
        u, v = s[0], s[1]
        out = [u * (1 - u), u - v + c]
        if len(s) == 3:
            p = self.p
            out.append(p["a_w"] * u - p["b_w"] * s[2] + p["s_w"])
        return torch.stack(out)

    def _node(self, G, c):
        """theta - phi(theta) / 2 = G of the implicit source, u then v."""
        u = 2 * G[0] / (0.5 + torch.sqrt(0.25 + 2 * G[0]))
        return torch.stack([u, (G[1] + 0.5 * (u + c)) / 1.5])

    def _sources(self, phi):
        return self.w[None, :, None] * phi[:, None]

    def step(self, f, c, first):
        s = f.sum(1)
        half = self.source == 3
        if half and not first:
            s = self._node(s, c)
            f = f + 0.5 * self._sources(self._kinetics(s, c))
        kin = self._kinetics(s, c) * (0.5 if half else 1.0)
        ET = self.E.T.to(f.dtype)
        flux = sum(B.to(f.dtype) @ (ET @ f[1 + k]) for k, B in enumerate(self.B)) * s[0]
        post = torch.stack([A.to(f.dtype) @ f[k] for k, A in enumerate(self.A)])
        chemo = 3 * self.w[:, None] * (self.E.to(f.dtype) @ flux)
        post = post + self._sources(kin)
        return self._stream(torch.cat([(post[0] + chemo)[None], post[1:]]))

    def theta(self, f, c):
        s = f.sum(1)
        s = self._node(s, c) if self.source == 3 else s
        return s[0] * self.fluid, s[1] * self.fluid

    def final(self, c):
        f = self.f0.to(c.dtype)
        with torch.no_grad():
            for n in range(self.steps):
                f = self.step(f, c, n == 0)
            return self.theta(f, c)

    def gradient(self):
        """u^N, v^N, dJ/dc, recomputing segments of the trajectory."""
        N = self.steps
        size = self.f0.numel() * 8
        seg = max(1, min(N, int(math.sqrt(N)) if N * size > 2e10 else N))
        kept, f = {}, self.f0
        with torch.no_grad():
            for n in range(N):
                if n % seg == 0:
                    kept[n] = f
                f = self.step(f, self.c, n == 0)
        f = f.detach().requires_grad_(True)
        c = self.c.clone().requires_grad_(True)
        uN, vN = self.theta(f, c)
        J = 0.5 * (((uN - self.target) * self.fluid) ** 2).sum() + 0.5 * self.p["alpha"] * (c * c).sum()
        lam, g = torch.autograd.grad(J, (f, c))
        for n0 in sorted(kept, reverse=True):
            states = [kept[n0]]
            with torch.no_grad():
                for n in range(n0, min(N, n0 + seg) - 1):
                    states.append(self.step(states[-1], self.c, n == 0))
            for n in range(min(N, n0 + seg) - 1, n0 - 1, -1):
                f = states.pop().requires_grad_(True)
                c = self.c.clone().requires_grad_(True)
                lam, gc = torch.autograd.grad(self.step(f, c, n == 0), (f, c), lam)
                g = g + gc
        return uN.detach(), vN.detach(), g * self.fluid, float(J.detach())


def _field(x, shape):
    return x.reshape(shape)


def _exact_network(params, x, in_scale=0.2, out_scale=0.1):
    """The four periodic convolutions, [B, h, w] in float64."""
    a = x[:, None] * in_scale
    for layer, (w, b) in enumerate(params):
        z = 0
        for ky in range(3):
            for kx in range(3):
                r = torch.roll(a, (1 - ky, 1 - kx), (2, 3))
                z = z + torch.tensordot(w[:, :, ky, kx], r, ([1], [1])).transpose(0, 1)
        z = z + b[None, :, None, None]
        a = torch.tanh(z) if layer < 3 else out_scale * z
    return a[:, 0]


def _exact_train(case, seed):
    s, e = int(seed) % 65536, case["crop"]
    x = _images(seed, case["pool"], case["size"], case["size"]).double()
    y = (0.02 * _images(seed + 1, case["pool"], case["size"], case["size"])).double()
    params = [tuple(torch.tensor(a, device=DEV).requires_grad_(True) for a in wb)
              for wb in _network(seed)]
    flat = [t for wb in params for t in wb]
    m, v = [torch.zeros_like(t) for t in flat], [torch.zeros_like(t) for t in flat]
    rng, losses, grads = np.random.default_rng(s), [], None
    span = np.arange(e)
    for k in range(case["steps"]):
        idx = rng.integers(0, case["pool"], case["batch"])
        oy, ox = (rng.integers(0, case["size"], case["batch"]) for _ in range(2))
        yy = torch.tensor((oy[:, None] + span) % case["size"], device=DEV)
        xx = torch.tensor((ox[:, None] + span) % case["size"], device=DEV)
        ii = torch.tensor(idx, device=DEV)
        at = (ii[:, None, None], yy[:, :, None], xx[:, None, :])
        # the hidden layers multiply bfloat16 copies of the masters
        low = [(w + (w.detach().bfloat16().double() - w.detach()), b) for w, b in params]
        d = (_exact_network(low, x[at]) - y[at])[:, 4:e - 4, 4:e - 4]
        loss = (d * d).mean()
        losses.append(float(loss.detach()))
        grads = torch.autograd.grad(loss, flat)
        lr = 2e-3 * max(0.5 * (1 + math.cos(math.pi * k / case["steps"])), 1e-3)
        with torch.no_grad():
            for t, g, a, b in zip(flat, grads, m, v):
                a.mul_(0.9).add_(0.1 * g)
                b.mul_(0.999).add_(0.001 * g * g)
                t.sub_(lr * (a / (1 - 0.9 ** (k + 1))) / ((b / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8))
    out = []
    for layer in range(4):
        out += [t.detach().reshape(-1) for t in params[layer]]
        out += [t.reshape(-1) for t in grads[2 * layer:2 * layer + 2]]
    return dict(params=out, loss=np.array([losses[0], losses[-1]]))


def _zeta_step(x, g):
    return min(1.0, 1.0 / float(g.abs().max()))


def exact(case, seed):
    k = case["kind"]
    if k == "train":
        return _exact_train(case, seed)
    if k == "score":
        params = [tuple(torch.tensor(a, device=DEV) for a in wb) for wb in _network(seed)]
        x = _images(seed, case["batch"], case["h"], case["w"]).double()
        return torch.cat([_exact_network(params, x[i:i + 1]) for i in range(case["batch"])])
    if k == "batch":
        js, each = [], []
        for i, c in enumerate(_batch_cases(case)):
            m = _Exact(_fields(c, seed * 100 + i), c["steps"])
            uN, _, g, J = m.gradient()
            js.append(J)
            each.append([_field(a, m.shape) for a in (g, uN, m.c - _zeta_step(m, g) * g)])
        return dict(J=np.array(js), each=each)
    if "nz" in case and case["nx"] * case["ny"] * case["nz"] > 5e6:
        return None
    m = _Exact(_fields(case, seed), case["steps"], case.get("source", 1))
    if k == "forward":
        uN, vN = m.final(m.c)
        J = 0.5 * float((((uN - m.target) * m.fluid) ** 2).sum()) + 0.5e-3 * float((m.c ** 2).sum())
        return dict(uN=_field(uN, m.shape), vN=_field(vN, m.shape), J=np.array(J))
    uN, vN, g, J = m.gradient()
    out = dict(grad=_field(g, m.shape), uN=_field(uN, m.shape), vN=_field(vN, m.shape))
    if k == "autograd":
        return out
    if case.get("op") == "lma":
        h = 1e-30
        P = m.final(m.c + 1j * h * g)[0].imag / h
        resid = (uN - m.target) * m.fluid
        zeta = float((resid * P).sum() + 1e-3 * (m.c * g).sum()) / float(
            (P * P).sum() + 1e-3 * (g * g).sum())
        out["tangent"] = _field(P, m.shape)
    else:
        zeta = _zeta_step(m, g)
        out["control"] = _field(m.c - zeta * g, m.shape)
    out["scalars"] = np.array([J, zeta])
    return out
