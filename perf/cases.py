"""Performance cases of the Nabla operators and the remap on one GPU.

Each case is one piece of work as a program using the library has it do:
a field (or wind, or cotangent) resident on the GPU goes through a public
call and the outputs come back whole.  Grid and level counts are those of the
tests, the benchmark and the batched workload (O32 x 10, O320, O640 and
O1280, 1, 19, 60, 91 and 137 levels); draw() spreads over the range between.

Meshes, remap tables and batched plans belong to the program, not to a call:
they are built once and kept, as a model keeps its grid.
"""

import functools
import math

import numpy as np
import torch

import paper_1908_07038_amd as pa

RADIUS = 6371220.0
DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
SIZES = {"f64": 8, "f32": 4, "bf16": 2}
GEOMETRY_BYTES = 104      # S_e and both ends of three edges, and V_i, per node (FP64)
LEVEL_CHOICES = (1, 19, 60, 91, 137)   # tracer depths of the batched workload

# op: (components in, elements read per node-level, elements written, flops per node-level)
OPS = {
    "gradient": (1, 1, 2, 30), "divergence": (2, 2, 1, 28), "curl": (2, 2, 1, 28), "laplacian": (1, 1, 1, 54),
    "gradient_adjoint": (2, 2, 1, 28), "divergence_adjoint": (1, 1, 2, 26), "curl_adjoint": (1, 1, 2, 26),
    "gradient_laplacian": (1, 1, 3, 84), "divergence_curl": (2, 2, 2, 56),
    "divergence_gradient_adjoint": (2, 2, 2, 56),
    # diagnostics of one field: gradient and Laplacian, divergence and gradient
    # adjoint of the gradient, divergence adjoint of the divergence
    "step": (1, 4, 7, 166),
    # differentiable gradient and Laplacian, forward and backward: reads the
    # field and both cotangents, writes both outputs and the input gradient
    "train": (1, 4, 4, 180),
    "conservation": (1, 1, 0, 3),
    "remap": (1, 0, 0, 5), "remap_adjoint": (1, 0, 0, 5),
    "batch": (1, 4, 6, 112),
}


def listed():
    return [
        # a small call, as in a first script or a test: launch latency
        dict(name="gradient_o32_l10_f64", op="gradient", N=32, L=10, dtype="f64"),
        # a surface field (log surface pressure): one level, tables dominate
        dict(name="gradient_o640_l1_f32", op="gradient", N=640, L=1, dtype="f32"),
        # a short column (soil, ocean waves, a coarse tracer): wind divergence
        dict(name="divergence_o640_l19_f32", op="divergence", N=640, L=19, dtype="f32"),
        # full-precision diffusion on a medium grid
        dict(name="laplacian_o320_l137_f64", op="laplacian", N=320, L=137, dtype="f64"),
        # diffusion of a field stored in 16 bits
        dict(name="laplacian_o640_l60_bf16", op="laplacian", N=640, L=60, dtype="bf16"),
        # divergence and vorticity of a wind stored in 16 bits
        dict(name="divcurl_o640_l91_bf16", op="divergence_curl", N=640, L=91, dtype="bf16"),
        # the benchmark's operators at its size
        dict(name="step_o1280_l137_f32", op="step", N=1280, L=137, dtype="f32"),
        # global mass of a tracer
        dict(name="mass_o1280_l137_f32", op="conservation", N=1280, L=137, dtype="f32"),
        # an optimisation or assimilation step through the differentiable form
        dict(name="train_o320_l60_f32", op="train", N=320, L=60, dtype="f32"),
        # many tracers of mixed depths in one plan
        dict(name="batch_o320_t16_f32", op="batch", N=320, L=0, dtype="f32", tracers=16, tseed=1005),
        # output to a regular Gaussian grid of half the resolution
        dict(name="remap_o1280_f640_l137_f32", op="remap", N=1280, L=137, dtype="f32", target="F640"),
        # backward of that interpolation, full precision
        dict(name="remap_adjoint_o640_f320_l91_f64", op="remap_adjoint", N=640, L=91, dtype="f64", target="F320"),
    ]


def draw(rng):
    """A case of the same ranges: any operator, O16..O640, 1..200 levels."""
    op = rng.choice(sorted(OPS))
    n = int(round(math.exp(rng.uniform(math.log(16), math.log(640)))))
    levels = int(round(math.exp(rng.uniform(0.0, math.log(200)))))
    dtype = rng.choice(("f64", "f32", "f32", "bf16"))
    if op in ("step", "train", "batch") and dtype == "bf16":
        dtype = "f32"      # chains keep 32 bits between operators; plans take f32 and f64
    case = dict(op=op, N=n, L=levels, dtype=dtype)
    if op in ("remap", "remap_adjoint"):
        case["target"] = rng.choice("FO") + str(max(4, int(n * rng.uniform(0.3, 1.0))))
    if op == "batch":
        case.update(N=min(n, 320), L=0, tracers=rng.randint(2, 16), tseed=rng.randrange(1 << 20))
    return case


# ---- what the program keeps ------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _mesh(n):
    return pa.Mesh(f"O{n}", radius=RADIUS, device=0)


@functools.lru_cache(maxsize=None)
def _remap(n, target):
    return pa.Remap(_mesh(n), target)


def _device():
    return torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")


@functools.lru_cache(maxsize=None)
def _xyz(n):
    return torch.from_numpy(_mesh(n).export_grid()["xyz"]).to(_device(), torch.float32)


def tracer_levels(case):
    return [int(v) for v in np.random.default_rng(case["tseed"]).choice(LEVEL_CHOICES, case["tracers"])]


# ---- inputs ------------------------------------------------------------------------

def _smooth(points, gen):
    """A smooth field of order 1: a few plane waves over the unit sphere."""
    k = torch.randn(12, 3, generator=gen) * 8.0
    phase = torch.rand(12, generator=gen) * (2 * math.pi)
    amp = torch.randn(12, generator=gen) * 0.4
    s = torch.zeros(points.shape[0], dtype=torch.float32, device=points.device)
    for q in range(12):
        s += float(amp[q]) * torch.sin(points @ k[q].to(points.device) + float(phase[q]))
    return s


def _field(points, levels, comps, dtype, gen, offset=0.0):
    """[points][levels] or [points][levels][2]: a smooth field whose amplitude
    grows with the level, an offset, and noise of 1e-3."""
    dev = points.device
    g = torch.Generator(device=dev).manual_seed(int(torch.randint(1 << 62, (1,), generator=gen)))
    shape = (points.shape[0], levels) + ((2,) if comps == 2 else ())
    work = torch.float64 if dtype == torch.float64 else torch.float32
    x = torch.randn(shape, generator=g, dtype=work, device=dev).mul_(1e-3)
    scale = 1.0 + 0.1 * torch.arange(levels, dtype=work, device=dev)
    for c in range(comps):
        part = x[..., c] if comps == 2 else x
        part.addcmul_(_smooth(points, gen).to(work)[:, None], scale[None, :])
    if offset:
        x.add_(offset)
    return x if x.dtype == dtype else x.to(dtype)


def prepare(case, seed):
    gen = torch.Generator().manual_seed(seed)
    op, n, levels, dtype = case["op"], case["N"], case["L"], DTYPES[case["dtype"]]
    m, xyz = _mesh(n), _xyz(n)
    state = dict(op=op, mesh=m)
    if op == "batch":
        tracers = []
        for nl in tracer_levels(case):
            f = _field(xyz, nl, 1, dtype, gen)
            uv = _field(xyz, nl, 2, dtype, gen)
            one = lambda: torch.empty_like(f)    # noqa: E731
            two = lambda: torch.empty_like(uv)   # noqa: E731
            tracers.append({"gradient": (f, two()), "divergence": (uv, one()),
                            "gradient_adjoint": (uv, one()), "divergence_adjoint": (f, two())})
        state.update(tracers=tracers, plan=pa.Batch(m, tracers))
        return state
    if op in ("remap", "remap_adjoint"):
        r = _remap(n, case["target"])
        state["remap"] = r
        if op == "remap":
            state["x"] = _field(xyz, levels, 1, dtype, gen)
        else:
            points = _target_xyz(n, case["target"])
            state["x"] = _field(points, levels, 1, dtype, gen)
        return state
    # a tracer's mass is of a positive quantity
    state["x"] = _field(xyz, levels, OPS[op][0], dtype, gen, offset=50.0 if op == "conservation" else 0.0)
    if op == "train":
        state["x"].requires_grad_(True)
        state["gbar"] = _field(xyz, levels, 2, dtype, gen)
        state["lbar"] = _field(xyz, levels, 1, dtype, gen)
    return state


@functools.lru_cache(maxsize=None)
def _target_xyz(n, target):
    return torch.from_numpy(_remap(n, target).export()["xyz"]).to(_device(), torch.float32)


# ---- one pass ----------------------------------------------------------------------

def run(state):
    op, m = state["op"], state["mesh"]
    if op == "batch":
        state["plan"].run()
        return [[t[name][1] for name in sorted(t)] for t in state["tracers"]]
    x = state["x"]
    if op == "step":
        g, lap = pa.gradient_laplacian(m, x)
        d, ft = pa.divergence_gradient_adjoint(m, g)
        return g, lap, d, ft, pa.divergence_adjoint(m, d)
    if op == "train":
        g, lap = pa.grad_lap(m, x)
        fbar, = torch.autograd.grad((g, lap), x, (state["gbar"], state["lbar"]))
        return g.detach(), lap.detach(), fbar
    if op == "remap":
        return state["remap"](x)
    if op == "remap_adjoint":
        return state["remap"].adjoint(x)
    return getattr(pa, op)(m, x)


def work(case):
    """Fields read once and written once, and the geometry (or the target's
    indices and weights) once."""
    op, n, es = case["op"], case["N"], SIZES[case["dtype"]]
    nodes = 4 * n * n + 36 * n
    if op in ("remap", "remap_adjoint"):
        k = int(case["target"][1:])
        points = 8 * k * k if case["target"][0] == "F" else 4 * k * k + 36 * k
        moved = (min(nodes, 3 * points) if op == "remap" else nodes) + points
        weights = 12 + 3 * (8 if es == 8 else 4)
        return dict(bytes=case["L"] * es * moved + weights * points, flops=OPS[op][3] * case["L"] * points)
    levels = sum(tracer_levels(case)) if op == "batch" else case["L"]
    _, read, written, flops = OPS[op]
    if op == "batch":
        read = 3           # the scalar field and the wind, each once
    if op == "step":
        read = 1           # what is computed on the way need not be read again
    geometry = 8 if op == "conservation" else GEOMETRY_BYTES
    out = 16 * levels if op == "conservation" else 0
    return dict(bytes=nodes * levels * es * (read + written) + geometry * nodes + out, flops=flops * nodes * levels)


# ---- the same in 64 bits ------------------------------------------------------------

class _Exact:
    """The operators in plain torch on the mesh's exported FP64 geometry: sums
    over each node's faces, blocks of levels at a time."""

    BLOCK = 8

    def __init__(self, n):
        m, dev = _mesh(n), _device()
        con, geo, grid = m.export_connectivity(), m.export_geometry(), m.export_grid()
        off = con["csr_off"]
        deg = np.diff(off)
        self.slots, v = int(deg.max()), m.nnodes
        owner = np.repeat(np.arange(v), deg)
        slot = np.arange(owner.size) - off[owner]
        nbr = np.tile(np.arange(v)[:, None], (1, self.slots))
        face = np.zeros((v, self.slots, 3))
        nbr[owner, slot] = con["nbr"]
        face[owner, slot] = con["sgn"][:, None] * geo["S"][con["eid"]]
        self.nbr = torch.from_numpy(nbr).to(dev)
        self.face = torch.from_numpy(face).to(dev)        # outward face vectors, zero past the degree
        self.vol = torch.from_numpy(geo["V"]).to(dev)
        self.basis = torch.from_numpy(geo["basis"]).to(dev)
        self.xyz = torch.from_numpy(grid["xyz"]).to(dev)

    def tangent(self, s):
        mid = self.xyz + self.xyz[self.nbr[:, s]]
        mid = mid / mid.norm(dim=1, keepdim=True)
        return torch.linalg.cross(mid, self.face[:, s])

    def _blocks(self, x, out_comps, one):
        v, levels = x.shape[:2]
        out = torch.empty((v, levels) + ((2,) if out_comps == 2 else ()), dtype=torch.float64, device=x.device)
        for k in range(0, levels, self.BLOCK):
            out[:, k:k + self.BLOCK] = one(x[:, k:k + self.BLOCK].double())
        return out

    def _to_local(self, parts):
        """Sum over slots of value [V][B] times vector [V][3], on (east, north)."""
        e = nn = 0
        for value, vec in parts:
            e = e + value * (vec * self.basis[:, 0]).sum(1)[:, None]
            nn = nn + value * (vec * self.basis[:, 1]).sum(1)[:, None]
        return torch.stack((e, nn), dim=2)

    def _dot(self, u, nodes, vec):
        """Wind (east, north) of the given nodes with a vector [V][3]."""
        b = self.basis if nodes is None else self.basis[nodes]
        w = u if nodes is None else u[nodes]
        return w[..., 0] * (b[:, 0] * vec).sum(1)[:, None] + w[..., 1] * (b[:, 1] * vec).sum(1)[:, None]

    def gradient(self, f):
        def one(x):
            return self._to_local((0.5 * (x[self.nbr[:, s]] - x), self.face[:, s] / self.vol[:, None])
                                  for s in range(self.slots))
        return self._blocks(f, 2, one)

    def _divergence(self, uv, vector):
        def one(u):
            out = 0
            for s in range(self.slots):
                a = vector(s)
                out = out + 0.5 * (self._dot(u, None, a) + self._dot(u, self.nbr[:, s], a))
            return out / self.vol[:, None]
        return self._blocks(uv, 1, one)

    def divergence(self, uv):
        return self._divergence(uv, lambda s: self.face[:, s])

    def curl(self, uv):
        return self._divergence(uv, self.tangent)

    def laplacian(self, f):
        return self.divergence(self.gradient(f))

    def gradient_adjoint(self, w):
        def one(u):
            scaled = u / self.vol[:, None, None]
            out = 0
            for s in range(self.slots):
                a = self.face[:, s]
                out = out - 0.5 * (self._dot(scaled, None, a) + self._dot(scaled, self.nbr[:, s], a))
            return out
        return self._blocks(w, 1, one)

    def _divergence_adjoint(self, d, vector):
        def one(x):
            scaled = x / self.vol[:, None]
            return self._to_local((0.5 * (scaled - scaled[self.nbr[:, s]]), vector(s)) for s in range(self.slots))
        return self._blocks(d, 2, one)

    def divergence_adjoint(self, d):
        return self._divergence_adjoint(d, lambda s: self.face[:, s])

    def curl_adjoint(self, z):
        return self._divergence_adjoint(z, self.tangent)


@functools.lru_cache(maxsize=1)
def _exact_mesh(n):
    return _Exact(n)


def _exact_remap(r, x, rows):
    """w0 f[n0] + w1 f[n1] + w2 f[n2] of each target point, or its transpose
    onto `rows` nodes."""
    t = r.export()
    nodes = torch.from_numpy(t["nodes"].astype(np.int64)).to(x.device)
    w = torch.from_numpy(t["weights"]).to(x.device)
    x = x.double()
    if rows is None:
        return sum(w[:, j, None] * x[nodes[:, j]] for j in range(3))
    out = torch.zeros((rows, x.shape[1]), dtype=torch.float64, device=x.device)
    for j in range(3):
        out.index_add_(0, nodes[:, j], w[:, j, None] * x)
    return out


def exact(case, seed):
    op, n = case["op"], case["N"]
    state = prepare(case, seed)
    if op in ("remap", "remap_adjoint"):
        return _exact_remap(state["remap"], state["x"], state["mesh"].nnodes if op == "remap_adjoint" else None)
    e = _exact_mesh(n)
    if op == "batch":
        return [[getattr(e, name)(t[name][0]) for name in sorted(t)] for t in state["tracers"]]
    x = state["x"].detach()
    if op == "step":
        g = e.gradient(x)
        d = e.divergence(g)
        return g, d, d, e.gradient_adjoint(g), e.divergence_adjoint(d)
    if op == "train":
        g = e.gradient(x)
        w = state["gbar"].double() + e.divergence_adjoint(state["lbar"])
        return g, e.divergence(g), e.gradient_adjoint(w)
    if op == "conservation":
        p = x.double() * e.vol[:, None]
        return p.sum(0), p.abs().sum(0)
    if op == "gradient_laplacian":
        g = e.gradient(x)
        return g, e.divergence(g)
    if op == "divergence_curl":
        return e.divergence(x), e.curl(x)
    if op == "divergence_gradient_adjoint":
        return e.divergence(x), e.gradient_adjoint(x)
    return getattr(e, op)(x)
