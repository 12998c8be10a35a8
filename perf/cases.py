"""The framework's work as its users have it done, case by case, for timing.

Every case makes seeded synthetic input on the GPU, keeps what a program would keep between calls (the
context or engine, its parameters, the direction table), and runs one pass through the public entry
points of ``paper_1804_06304_amd.snk``. The kinds:

  segment   one volume or image whole: load it (borrowed on the device), seed, evolve, finalise, read
  block     a slice of a run on a volume already smoothed: seed, evolve a few iterations, read
  smooth    the low-pass alone, read back on the device
  lattice   the unattended workflow: lattice seeds, evolution with culling, finalise, read
  star      contours with one radius per direction
  sums      exact lattice sums instead of Monte-Carlo samples
  gradient  centre force in its image-gradient form
  repel     two seeds per nucleus with soft repulsion
  batch     an engine evolves many volumes of uneven size in one run
  served    an engine steps a queue of tile requests to completion

``exact`` evaluates the same iterations in 64 bits with torch alone.
"""
from __future__ import annotations

import ctypes
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1804_06304_amd import snk

SEED = 0x1804063040000000
DTYPES = {"u8": torch.uint8, "u16": torch.uint16, "f32": torch.float32}


# ------------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------------

def _case(name, kind, shape, n, **kw):
    """shape (nx, ny, nz); n nuclei. active: the share of contour-iterations that contours still
    evolving take (the others have converged or were culled), for work()."""
    c = {"name": name, "kind": kind, "nx": shape[0], "ny": shape[1], "nz": shape[2], "n": n, "hz": 2.0,
         "dtype": "u16", "D": 642, "M": 64, "iters": 500, "sigma": 1.0, "jobs": 1, "active": 1.0}
    c.update(kw)
    return c


def listed():
    return [
        # a handful of cells in a small stack (an interactive click, a unit of a script): latency
        _case("few_cells", "segment", (64, 64, 64), 8, hz=1.0, dtype="u8", D=162, M=32, iters=100),
        # the benchmark's slab whole: a confocal stack with 2,000 nuclei, run to convergence
        _case("slab", "segment", (512, 512, 128), 2000, active=0.75),
        # one slice of a longer run on the slab (progress shown or state saved between slices)
        _case("slab_slice", "block", (512, 512, 128), 2000, iters=25),
        # the benchmark's 2D image: a whole-slide tile with 40,000 cells
        _case("plane", "segment", (8192, 8192, 1), 40000, hz=1.0, dtype="u8", D=64, M=16, iters=300),
        # an odd-sized float stack smoothed with a wider filter than the benchmark's
        _case("smooth_odd", "smooth", (411, 387, 131), 0, dtype="f32", sigma=1.6),
        # nothing known about the cells: lattice seeds on the slab, culling every 25 iterations
        _case("lattice", "lattice", (512, 512, 128), 2000, active=0.1),
        # shapes instead of spheres: per-direction radii on a stack of 600 nuclei
        _case("star", "star", (256, 256, 128), 600, iters=60),
        # the deterministic sums, for users who want no random numbers
        _case("exact_sums", "sums", (256, 256, 128), 600, iters=60),
        # the variance-reduced centre force with half the rays
        _case("gradient_form", "gradient", (384, 384, 96), 1200, M=32, iters=100),
        # doubled seeds pushed apart, neighbours refreshed every 5 iterations
        _case("repulsion", "repel", (256, 256, 128), 600, iters=60),
        # uneven subvolumes in one engine run (edges 32 up to the case's nx, two sampling classes)
        _case("batch", "batch", (112, 112, 112), 300, iters=120, jobs=24),
        # tile requests through the serving loop, 25 iterations a step (edges 64 up to the case's nx)
        _case("served", "served", (160, 160, 160), 300, D=162, M=32, iters=200, jobs=10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the same kinds; sizes spread over their logarithm, odd ones among them."""
    kind = rng.choice(["segment", "segment", "plane", "block", "smooth", "lattice", "star", "sums", "gradient", "repel",
                       "batch", "served"])
    shape = (_log(rng, 64, 512), _log(rng, 64, 512), _log(rng, 24, 128))
    room = shape[0] * shape[1] * shape[2] * 2.0 / 20.0 ** 3
    n = max(4, int(room * rng.uniform(0.1, 0.45)))
    D, M = rng.choice([(162, 32), (642, 64)])
    kw = {"hz": rng.choice([1.0, 2.0, 2.0, 2.5]), "dtype": rng.choice(["u8", "u16", "u16", "f32"]), "D": D, "M": M}
    if kind == "plane":
        nx, ny = _log(rng, 256, 8192), _log(rng, 256, 8192)
        kw.update(hz=1.0, D=64, M=16, iters=rng.randint(100, 300))
        return _unnamed(_case("", "segment", (nx, ny, 1), max(8, int(nx * ny / 1700 * rng.uniform(0.2, 1.0))), **kw))
    if kind == "segment":
        return _unnamed(_case("", kind, shape, n, iters=rng.randint(100, 500), active=0.8, **kw))
    if kind == "block":
        return _unnamed(_case("", kind, shape, n, iters=rng.randint(5, 40), **kw))
    if kind == "smooth":
        kw.update(sigma=rng.choice([0.7, 1.0, 1.6, 2.2]))
        return _unnamed(_case("", kind, shape, 0, **kw))
    if kind == "lattice":
        return _unnamed(_case("", kind, shape, n, iters=rng.randint(100, 500), active=0.15, **kw))
    if kind in ("batch", "served"):
        top = _log(rng, 72, 128)
        kw.update(hz=2.0, D=162, M=32, iters=rng.randint(50, 200), jobs=rng.randint(2, 24))
        return _unnamed(_case("", kind, (top, top, top), 200, **kw))
    small = tuple(min(s, m) for s, m in zip(shape, (256, 256, 128)))
    room = small[0] * small[1] * small[2] * 2.0 / 20.0 ** 3
    return _unnamed(_case("", kind, small, max(4, int(room * rng.uniform(0.1, 0.3))), iters=rng.randint(10, 60), **kw))


def _unnamed(c):
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------

def _icosphere(subdiv):
    """10 * 4**subdiv + 2 unit vectors: the icosahedron, each face split into four `subdiv` times."""
    g = (1.0 + math.sqrt(5.0)) / 2.0
    v = [np.array(p) / math.sqrt(1 + g * g) for a in (-1.0, 1.0) for b in (-g, g) for p in ((0, a, b), (a, b, 0), (b, 0, a))]
    edge = 2.0 / math.sqrt(1 + g * g) + 1e-9
    near = [[np.linalg.norm(p - q) < edge for q in v] for p in v]
    faces = [(i, j, k) for i in range(12) for j in range(i) for k in range(j) if near[i][j] and near[j][k] and near[i][k]]
    for _ in range(subdiv):
        mids, split = {}, []
        for a, b, c in faces:
            m = []
            for i, j in ((a, b), (b, c), (c, a)):
                key = (min(i, j), max(i, j))
                if key not in mids:
                    p = v[i] + v[j]
                    v.append(p / np.linalg.norm(p))
                    mids[key] = len(v) - 1
                m.append(mids[key])
            split += [(a, m[0], m[2]), (b, m[1], m[0]), (c, m[2], m[1]), tuple(m)]
        faces = split
    return np.stack(v).astype(np.float32)


def _directions(dim, D):
    if dim == 2:
        a = 2.0 * np.pi * np.arange(D) / D
        return np.stack([np.cos(a), np.sin(a)], axis=1).astype(np.float32)
    return _icosphere({12: 0, 42: 1, 162: 2, 642: 3}[D])


def _params(c, key):
    dim = 2 if c["nz"] == 1 else 3
    lo, hi = (20.0, 160.0) if c["dtype"] == "u8" else (100.0, 900.0)
    r0 = 2.0 ** 0.5 * 8.0 if dim == 2 else 2.0 ** (1.0 / 3.0) * 6.5
    if c["kind"] == "segment" and c["nx"] == 64:
        r0 = 2.0 ** (1.0 / 3.0) * 5.5
    return SimpleNamespace(dim=dim, spacing=(1.0, 1.0, c["hz"]), sigma_pre=c["sigma"], i_offset=lo, i_scale=1.0 / hi,
                           dR=0.75 if c["D"] == 642 else 1.0, eps0=8.0, r_min=0.0, r_max=3.0 * r0, r_init=r0,
                           n_dirs=c["D"], n_rays=c["M"], n_radial=16, seed=SEED + key % 1000003, conv_tol=1e-3,
                           conv_window=10, e0=-0.08 if dim == 2 else -0.05,
                           flags={"sums": 2, "gradient": 4}.get(c["kind"], 0))


def _rotations(n, gen):
    q = torch.randn(n, 4, device="cuda", generator=gen)
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z),
                        1 - 2 * (x * x + z * z), 2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x),
                        1 - 2 * (x * x + y * y)], 1).reshape(n, 3, 3)


def _cells(shape, hz, n, dtype, gen):
    """A raw volume [z][y][x] with about n bright ellipsoids of random orientation (semi-axes 3..10
    physical units; 4..12 and round in 2D) on a jittered grid, blurred by the optics, with shot noise
    (u16, f32) or Gaussian noise (u8); and the cells' centres."""
    nx, ny, nz = shape
    dim = 2 if nz == 1 else 3
    h = torch.tensor([1.0, 1.0, hz], device="cuda")
    ext = torch.tensor([nx - 1.0, ny - 1.0, (nz - 1.0) * hz], device="cuda")
    lo, hi = (4.0, 12.0) if dim == 2 else (3.0, min(10.0, 0.3 * float(ext.min())))
    cells = [max(1, int(float(e) // (1.75 * hi))) for e in ext]
    if dim == 2:
        cells[2] = 1
    total = cells[0] * cells[1] * cells[2]
    pick = torch.randperm(total, device="cuda", generator=gen)[: max(1, min(n, total))]
    m = len(pick)
    at = torch.stack([pick % cells[0], pick // cells[0] % cells[1], pick // (cells[0] * cells[1])], 1).float()
    pitch = ext / torch.tensor(cells, device="cuda")
    cen = (at + 0.5 + 0.3 * (torch.rand(m, 3, device="cuda", generator=gen) - 0.5)) * pitch
    axes = lo + (hi - lo) * torch.rand(m, 3, device="cuda", generator=gen)
    rot = _rotations(m, gen)
    if dim == 2:
        cen[:, 2] = 0.0
        axes[:, 2] = 1.0
        rot = torch.eye(3, device="cuda").expand(m, 3, 3)
    half = [int(math.ceil((hi + 1.0) / float(h[a]))) if a < dim else 0 for a in range(3)]
    grid = torch.stack(torch.meshgrid(*(torch.arange(-k, k + 1, device="cuda") for k in half), indexing="ij"), -1).reshape(-1, 3)
    cov = torch.zeros(nx * ny * nz, device="cuda")
    top = torch.tensor([nx - 1, ny - 1, nz - 1], device="cuda")
    for b in range(0, m, 1024):
        c, ax, rm = cen[b:b + 1024], axes[b:b + 1024], rot[b:b + 1024]
        v = torch.round(c / h).long()[:, None, :] + grid
        q = torch.matmul((v * h - c[:, None, :]), rm) / ax[:, None, :]
        edge = (1.0 - q[..., :dim].norm(dim=-1)) * ax[:, None, :dim].amin(-1) + 0.5
        ok = ((v >= 0) & (v <= top)).all(-1) & (edge > 0)
        idx = (v[..., 2] * ny + v[..., 1]) * nx + v[..., 0]
        cov.scatter_reduce_(0, idx[ok], edge[ok].clamp(max=1.0), "amax")
    cov = cov.reshape(nz, ny, nx)
    taps = torch.exp(-torch.arange(-4, 5, dtype=torch.float64) ** 2 / (2 * 1.2 ** 2))
    taps = (taps / taps.sum()).tolist()
    for a in range(3 - dim, 3):
        idx = torch.arange(cov.shape[a], device="cuda")
        cov = sum(w * cov.index_select(a, (idx + k - 4).clamp(0, cov.shape[a] - 1)) for k, w in enumerate(taps))
    if dtype == "u8":
        raw = (20.0 + 160.0 * cov + 8.0 * torch.randn(cov.shape, device="cuda", generator=gen)).round().clamp(0, 255)
    else:
        gain = 1.0 - 0.3 * torch.arange(nx, device="cuda") / max(nx - 1, 1)
        raw = torch.poisson((100.0 + 900.0 * cov) * gain, generator=gen).clamp(max=65535)
    raw = raw.to(torch.int32).to(DTYPES[dtype]) if dtype != "f32" else raw
    return raw.contiguous(), cen.double().cpu().numpy()


def _job(c, seed, shape, n):
    """One volume with jittered seeds."""
    gen = torch.Generator("cuda")
    gen.manual_seed(seed)
    raw, cen = _cells(shape, c["hz"], n, c["dtype"], gen)
    rng = np.random.default_rng(seed)
    h = np.array([1.0, 1.0, c["hz"]])
    dim = 2 if shape[2] == 1 else 3
    if c["kind"] == "repel":
        cen = np.repeat(cen, 2, axis=0)
    jit = rng.uniform(-1.0, 1.0, size=cen.shape) * h * (1.5 if c["kind"] == "repel" else 1.0)
    jit[:, dim:] = 0.0
    seeds = np.clip(cen + jit, 0.0, (np.array(shape) - 1) * h)
    return raw, seeds, np.arange(len(seeds), dtype=np.uint32)


def _jobs(c, seed):
    rng = np.random.default_rng(c["jobs"])   # edges and counts belong to the case, the voxels to the seed
    lo = 32 if c["kind"] == "batch" else 64
    out = []
    for j in range(c["jobs"]):
        e = int(rng.integers(lo, c["nx"] + 1))
        p = _params(c, seed)
        if c["kind"] == "batch" and c["D"] == 642 and j % 2:   # two classes of sampling in one batch
            p.n_dirs, p.n_rays = 162, 32
        n = max(2, int(min(c["n"], 0.3 * e ** 3 * c["hz"] / 1150.0) * rng.uniform(0.3, 1.0)))
        out.append((p,) + _job(c, seed * 64 + j, (e, e, e), n))
    return out


def prepare(case, seed):
    c = case
    s = SimpleNamespace(c=c)
    stream = torch.cuda.current_stream()
    if c["kind"] in ("batch", "served"):
        s.jobs = [(snk.to_params(p), _directions(3, p.n_dirs), raw, seeds, ids) for p, raw, seeds, ids in _jobs(c, seed)]
        s.engine = snk.Engine(0, torch.cuda.Stream(), 64 << 30)
        # the shape a program keeps from an earlier tuning, so that its results replay bit for bit
        s.engine.set_launch(128, 2, 0, 0)
        s.engine.set_tile(4224 if c["kind"] == "batch" else 0, 0)
        return s
    s.p = _params(c, seed)
    s.raw, s.seeds, s.ids = _job(c, seed, (c["nx"], c["ny"], c["nz"]), max(c["n"], 1))
    s.ctx = snk.Context(0, stream)
    s.ctx.set_params(s.p)
    s.ctx.set_directions(_directions(s.p.dim, c["D"]))
    s.ctx.load_volume(s.raw)
    if c["kind"] == "lattice":
        s.ctx.set_cull(s.p.e0 / 4, False)
    if c["kind"] == "star":
        s.ctx.set_star(0.3)
    if c["kind"] == "repel":
        s.ctx.set_repulsion(0.1, 5)
    if c["kind"] == "smooth":
        s.out = torch.empty(s.raw.shape, dtype=torch.float32, device="cuda")
    elif c["kind"] != "segment":
        s.ctx.prepass()
    return s


# ------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------

def run(s):
    c = s.c
    kind, it = c["kind"], c["iters"]
    if kind == "batch":
        ids = [s.engine.submit(p, d, raw, seeds, ids=i, n_iter=it) for p, d, raw, seeds, i in s.jobs]
        s.engine.run()
        return _collect(s.engine, ids)
    if kind == "served":
        ids = [s.engine.submit(p, d, raw, seeds, ids=i, n_iter=it) for p, d, raw, seeds, i in s.jobs]
        left = len(ids)
        while left:
            left -= s.engine.step(25)
        s.engine.poll()
        return _collect(s.engine, ids)
    if kind == "smooth":
        s.ctx.load_volume(s.raw)
        s.ctx.prepass()
        code = snk.load().snk_read_volume(s.ctx.h, ctypes.c_void_p(s.out.data_ptr()), 1)
        if code:
            raise snk.SnkError(code, s.ctx.last_error())
        return s.out
    if kind == "lattice":
        s.ctx.seed_lattice(0.0)
        s.ctx.evolve_cull(it, 25, 50)
        s.ctx.finalize()
        return s.ctx.read()
    if kind == "segment":
        s.ctx.load_volume(s.raw)
    s.ctx.load_seeds(s.seeds, ids=s.ids)
    s.ctx.evolve(it)
    if kind == "block":
        out = s.ctx.get_state()
        out["e_mc"] = s.ctx.read()["e_mc"]
        return out
    s.ctx.finalize()
    out = s.ctx.read()
    if kind == "star":
        out["star_radii"] = s.ctx.get_star_radii()
    return out


def _collect(engine, ids):
    """The jobs' results in order, end to end; each job is released as a program does once it has read it."""
    parts = []
    for j in ids:
        parts.append(engine.read(j))
        engine.release(j)
    return {k: np.concatenate([p[k] for p in parts]) for k in parts[0]}


def work(case):
    """Raw voxels read once, results written once; per sample point of a contour-iteration the
    position, interpolation and sums (47 flops in 3D, 29 in 2D), per lattice point of the exact sums
    its distance, weight and sums (30), per voxel of the low-pass a multiply-add per tap and axis."""
    c = case
    size = {"u8": 1, "u16": 2, "f32": 4}[c["dtype"]]
    dim = 2 if c["nz"] == 1 else 3
    vox = c["nx"] * c["ny"] * c["nz"]
    taps = sum(2 * (2 * math.ceil(3 * c["sigma"] / (c["hz"] if a == 2 else 1.0)) + 1) for a in range(dim))
    if c["kind"] == "smooth":
        return {"bytes": vox * (size + 4), "flops": vox * taps}
    n = c["n"]
    if c["kind"] in ("batch", "served"):
        lo = 32 if c["kind"] == "batch" else 64
        mean = 0.25 * (c["nx"] ** 4 - lo ** 4) / max(c["nx"] - lo, 1)   # mean edge cubed over U[lo, nx]
        vox = mean * c["jobs"]
        n = c["jobs"] * 0.65 * min(c["n"], 0.3 * mean * c["hz"] / 1150.0)
    if c["kind"] == "lattice":
        pitch = math.sqrt(1.5) * 2.0 ** (1.0 / 3.0) * 6.5
        n = (c["nx"] / pitch) * (c["ny"] / pitch) * (c["nz"] * c["hz"] / pitch)
    if c["kind"] == "repel":
        n *= 2
    points = 1100.0 / c["hz"] * 30 if c["kind"] == "sums" else c["M"] * 16 * (47 if dim == 3 else 29)
    smooth = c["kind"] in ("segment", "batch", "served")
    return {"bytes": vox * size + n * 42, "flops": n * c["iters"] * c["active"] * points + (vox * taps if smooth else 0)}


# ------------------------------------------------------------------------------------------------
# the same in 64 bits
# ------------------------------------------------------------------------------------------------

def exact(case, seed):
    """What run() returns in 64 bits, None for whole-number outputs. None for the culled lattice (62,500
    contours take minutes), for a 2D image's 40,000 contours over hundreds of iterations and for more
    volumes than about 20 seconds allow."""
    c = case
    kind = c["kind"]
    if kind == "lattice" or c["nz"] == 1 and c["n"] * c["iters"] > 2_000_000:
        return None
    if kind in ("batch", "served"):
        if c["jobs"] * c["iters"] > 3000:
            return None
        parts = [_exact_run(c, p, raw, seeds, ids) for p, raw, seeds, ids in _jobs(c, seed)]
        return {k: None if parts[0][k] is None else np.concatenate([p[k] for p in parts]) for k in parts[0]}
    p = _params(c, seed)
    raw, seeds, ids = _job(c, seed, (c["nx"], c["ny"], c["nz"]), max(c["n"], 1))
    if kind == "smooth":
        return _smooth64(p, raw)
    return _exact_run(c, p, raw, seeds, ids)


def _smooth64(p, raw):
    J = (raw.to(torch.float64) - p.i_offset) * p.i_scale
    for a in range(3):
        axis = 2 - a
        sig = p.sigma_pre / p.spacing[a]
        if J.shape[axis] == 1 or sig <= 0 or a >= p.dim:
            continue
        r = math.ceil(3 * sig)
        w = np.exp(-np.arange(-r, r + 1) ** 2 / (2 * sig * sig))
        w /= w.sum()
        idx = torch.arange(J.shape[axis], device="cuda")
        J = sum(float(w[k + r]) * J.index_select(axis, (idx + k).clamp(0, J.shape[axis] - 1)) for k in range(-r, r + 1))
    return J


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors holding 32-bit words."""
    M0, M1, mask = 0xD2511F53, 0xCD9E8D57, 0xFFFFFFFF
    k0, k1 = seed & mask, seed >> 32 & mask

    def mul(m, x):   # 32 x 32 -> (high, low) without overflowing 64 signed bits
        lo, hi = (m & 0xFFFF) * x, (m >> 16) * x
        t = (lo >> 16) + (hi & 0xFFFF)
        return (hi >> 16) + (t >> 16), (t << 16 | lo & 0xFFFF) & mask

    for _ in range(10):
        h0, l0 = mul(M0, c0)
        h1, l1 = mul(M1, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = k0 + 0x9E3779B9 & mask, k1 + 0xBB67AE85 & mask
    return c0, c1, c2, c3


def _unit(x):
    return ((x >> 9) * 2 + 1).double() * 2.0 ** -24


class _Field:
    """The smoothed volume, read at physical points by clamped (bi/tri)linear interpolation."""

    def __init__(self, p, J):
        self.p, self.J = p, J.reshape(-1)
        self.n = [J.shape[2], J.shape[1], J.shape[0]]
        self.stride = [1, self.n[0], self.n[0] * self.n[1]]

    def at(self, x, grad=False):
        """x: dim tensors of physical coordinates -> value (and the physical gradient)."""
        dim = self.p.dim
        base, f, live = 0, [], []
        for a in range(dim):
            v = x[a] / self.p.spacing[a]
            live.append(((v >= 0) & (v <= self.n[a] - 1)).double())
            v = v.clamp(0, self.n[a] - 1)
            i = v.floor().clamp(max=self.n[a] - 2)
            f.append(v - i)
            base = base + i.long() * self.stride[a]
        val, g = 0.0, [0.0] * dim
        for corner in range(2 ** dim):
            bits = [corner >> a & 1 for a in range(dim)]
            J = self.J[base + sum(b * s for b, s in zip(bits, self.stride))]
            w = [f[a] if bits[a] else 1 - f[a] for a in range(dim)]
            val = val + math.prod(w) * J
            if grad:
                for a in range(dim):
                    others = math.prod([w[b] for b in range(dim) if b != a])
                    g[a] = g[a] + (1 if bits[a] else -1) * others * J
        return (val, [g[a] * live[a] / self.p.spacing[a] for a in range(dim)]) if grad else val

    def voxel(self, idx):
        """J at integer voxels, clamped to the volume."""
        return self.J[sum(idx[a].clamp(0, self.n[a] - 1) * self.stride[a] for a in range(self.p.dim))]


def _weights(p, r, R):
    """S, dS/dr and dS/dR at distance r for radius R (four half-open regions)."""
    rho = 2.0 ** (-1.0 / p.dim)
    a, dr = rho * R, rho * p.dR
    inner = (r >= a - dr / 2) & (r < a + dr / 2)
    outer = (r >= R - p.dR / 2) & (r < R + p.dR / 2)
    z = torch.zeros_like(r)
    S = torch.where(r < a - dr / 2, z - 1, torch.where(inner, 2 * (r - a) / dr, torch.where(
        r < R - p.dR / 2, z + 1, torch.where(outer, 0.5 - (r - R) / p.dR, z))))
    Sr = torch.where(inner, z + 2 / dr, torch.where(outer, z - 1 / p.dR, z))
    SR = torch.where(inner, z - rho * 2 / dr, torch.where(outer, z + 1 / p.dR, z))
    return S, Sr, SR


def _rays(p, dirs, n, ids, rotate=True):
    """Pair directions (contours, pairs, dim), table rows and jitters of iteration n (per contour)."""
    MH = p.n_rays // 2
    m = torch.arange(MH, device="cuda")[None, :]
    one = torch.ones_like(ids)[:, None]
    x = _philox(m * one, n[:, None] * one, ids[:, None] * torch.ones_like(m), torch.ones_like(m) * one, p.seed)
    k, xi = x[0] * p.n_dirs >> 32, _unit(x[1])
    u = dirs[k]
    if rotate:
        r = [_unit(v) for v in _philox(torch.zeros_like(ids), n, ids, torch.zeros_like(ids), p.seed)]
        if p.dim == 2:
            c, s = torch.cos(2 * math.pi * r[0]), torch.sin(2 * math.pi * r[0])
            Q = torch.stack([c, -s, s, c], 1).reshape(-1, 2, 2)
        else:   # Shoemake's uniform quaternion
            a, b = (1 - r[0]).sqrt(), r[0].sqrt()
            x, y = a * torch.sin(2 * math.pi * r[1]), a * torch.cos(2 * math.pi * r[1])
            z, w = b * torch.sin(2 * math.pi * r[2]), b * torch.cos(2 * math.pi * r[2])
            Q = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z),
                             1 - 2 * (x * x + z * z), 2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x),
                             1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)
        u = (Q[:, None] * u[:, :, None, :]).sum(-1)
    return u, k, xi


def _mc_sums(p, field, dirs, c, R, n, ids):
    """A, B_R, B_c of one Monte-Carlo iteration."""
    u, _, xi = _rays(p, dirs, n, ids)
    L = p.n_radial
    smax = R + p.dR / 2
    s = smax[:, None, None] * ((torch.arange(L, device="cuda") + xi[..., None]) / L) ** (1.0 / p.dim)
    S, Sr, SR = _weights(p, s, R[:, None, None])
    V = (4 * math.pi / 3 if p.dim == 3 else math.pi) * smax ** p.dim / (p.n_rays * L)
    A = B = 0.0
    Bc = [0.0] * p.dim
    for sign in (1.0, -1.0):
        x = [c[:, a, None, None] + sign * s * u[..., a, None] for a in range(p.dim)]
        if p.flags & 4:
            I, g = field.at(x, True)
        else:
            I = field.at(x)
        A, B = A + (S * I).sum((1, 2)), B + (SR * I).sum((1, 2))
        for a in range(p.dim):
            Bc[a] = Bc[a] + ((S * g[a]) if p.flags & 4 else -Sr * I * sign * u[..., a, None]).sum((1, 2))
    return V * A, V * B, torch.stack(Bc, 1) * V[:, None]


def _lattice(p, field, c, R, want):
    """Sums over the lattice points within R + dR/2 of the centre: "E" or (A, B_R, B_c)."""
    out = []
    h = torch.tensor(p.spacing[: p.dim], dtype=torch.float64, device="cuda")
    for b in range(0, len(R), 64):
        cc, RR = c[b:b + 64, : p.dim], R[b:b + 64]
        half = [int(v) + 1 for v in torch.ceil((RR.max() + p.dR / 2) / h).tolist()]
        grid = torch.stack(torch.meshgrid(*(torch.arange(-k, k + 1, device="cuda") for k in half), indexing="ij"), -1)
        k = torch.round(cc / h).long()[:, None, :] + grid.reshape(-1, p.dim)
        d = k * h - cc[:, None, :]
        r = d.norm(dim=-1)
        S, Sr, SR = _weights(p, r, RR[:, None])
        w = math.prod(p.spacing[: p.dim]) * field.voxel(k.unbind(-1)) * (r < RR[:, None] + p.dR / 2)
        A = (S * w).sum(1)
        if want == "E":
            out.append(A / (2 * RR) ** p.dim)
        else:
            g = -Sr * w / r.clamp(min=1e-300)
            out.append(torch.cat([A[:, None], (SR * w).sum(1, keepdim=True), (g[..., None] * d).sum(1)], 1))
    return torch.cat(out)


def _repulsion(p, c, R, snap):
    """Gradient of sum (1 - t)^2 over the live contours of the snapshot, t = |c - c_j| / (rho (R + R_j))."""
    cs, Rs, live = snap
    d = c[:, None, :] - cs[None]
    dist = d.norm(dim=-1)
    sum_R = R[:, None] + Rs[None]
    span = 2.0 ** (-1.0 / p.dim) * sum_R
    t = dist / span
    at0 = torch.norm(cs[:, None] - cs[None], dim=-1) < 2.0 ** (-1.0 / p.dim) * (Rs[:, None] + Rs[None])
    on = (t < 1) & live[None] & at0 & ~torch.eye(len(R), dtype=torch.bool, device="cuda")
    f = torch.where(on & (dist > 0), -2 * (1 - t) / (dist * span).clamp(min=1e-300), torch.zeros_like(t))
    return (f[..., None] * d).sum(1), torch.where(on, 2 * (1 - t) * t / sum_R, torch.zeros_like(t)).sum(1)


def _exact_run(c, p, raw, seeds, ids):
    field = _Field(p, _smooth64(p, raw))
    dim = p.dim
    dirs = torch.from_numpy(_directions(dim, p.n_dirs)).cuda().double()
    h = torch.tensor(p.spacing[:dim], dtype=torch.float64, device="cuda")
    cen = torch.from_numpy(seeds[:, :dim].copy()).cuda()
    ids = torch.from_numpy(ids.astype(np.int64)).cuda()
    rho = 2.0 ** (-1.0 / dim)
    r_lo = max(p.r_min, p.dR * (1 + rho) / (2 * (1 - rho)))
    R = torch.full((len(ids),), min(max(p.r_init, r_lo), p.r_max), dtype=torch.float64, device="cuda")
    top = (torch.tensor(field.n[:dim], device="cuda") - 1) * h
    n = torch.zeros_like(ids)
    on = ((cen >= 0) & (cen <= top)).all(1)
    streak = torch.zeros_like(ids)
    E = torch.zeros_like(R)
    star = _StarTables(dirs) if c["kind"] == "star" else None
    Rk = R[:, None].repeat(1, p.n_dirs) if star else None
    converged = torch.zeros_like(on)
    snap = None
    for it in range(c["iters"]):
        if c["kind"] == "repel" and it % 5 == 0:
            snap = (cen.clone(), R.clone(), on | converged)
        if not bool(on.any()):
            break
        w = on.nonzero()[:, 0]
        n[w] += 1
        eps = p.eps0 / n[w].double().sqrt()
        if star:
            e, gc, Rn = star.step(p, field, dirs, cen[w], Rk[w], n[w], ids[w], eps, 0.3)
            Rn = Rn.clamp(r_lo, p.r_max)
            move = (Rn - Rk[w]).abs().amax(1)
            Rk[w], R[w] = Rn, Rn.mean(1)
            dc = -eps[:, None] / 2 * gc
        else:
            RR = R[w]
            if p.flags & 2:
                sums = _lattice(p, field, cen[w], RR, "sums")
                A, B, Bc = sums[:, 0], sums[:, 1], sums[:, 2:]
            else:
                A, B, Bc = _mc_sums(p, field, dirs, cen[w], RR, n[w], ids[w])
            norm = (2 * RR) ** dim
            e = A / norm
            gR, gc = (B - dim / RR * A) / norm, Bc / norm[:, None]
            if snap:
                # every contour's pairs, the rows of those still moving taken
                pc, pR = _repulsion(p, cen, R, snap)
                gR, gc = gR + 0.1 * pR[w], gc + 0.1 * pc[w]
            Rn = (RR - eps / 2 * gR).clamp(r_lo, p.r_max)
            move = (Rn - RR).abs()
            R[w] = Rn
            dc = -eps[:, None] / 2 * gc
        E[w] = e
        cen[w] += dc
        small = (move < p.conv_tol) & (dc.norm(dim=1) < p.conv_tol)
        inside = ((cen[w] >= 0) & (cen[w] <= top)).all(1)
        streak[w] = torch.where(small, streak[w] + 1, torch.zeros_like(streak[w]))
        done = streak[w] >= p.conv_window
        converged[w] = inside & done
        on[w] = inside & ~done
    out = np.zeros((len(ids), 3))
    out[:, :dim] = cen.cpu().numpy()
    if c["kind"] == "block":
        return {"centers": out, "radii": R, "iters": None, "status": None, "streak": None, "e_mc": E}
    got = {"radii": R.cpu().numpy(), "centers": out, "e_mc": E.cpu().numpy(), "iters": None, "status": None, "keep": None,
           "e_vox": (E if star else _lattice(p, field, cen, R, "E")).cpu().numpy()}
    if star:
        got["star_radii"] = Rk.cpu().numpy()
    return got


class _StarTables:
    """Antipodes and the symmetric six-nearest (two in 2D) neighbour graph of a direction table."""

    def __init__(self, dirs):
        dots = dirs @ dirs.T
        self.anti = dots.argmin(1)
        deg = 6 if dirs.shape[1] == 3 else 2
        near = torch.zeros_like(dots, dtype=torch.bool)
        left = dots - 4 * torch.eye(len(dirs), dtype=dots.dtype, device=dots.device)
        rows = torch.arange(len(dirs), device=dots.device)
        for _ in range(deg):   # dot products within 1e-6 tie, the lower index first
            j = (left > left.amax(1, keepdim=True) - 1e-6).int().argmax(1)
            near[rows, j] = True
            left[rows, j] = -9.0
        near |= near.T.clone()
        self.mean = near.double() / near.sum(1, keepdim=True)

    def step(self, p, field, dirs, c, Rk, n, ids, eps, smooth):
        _, k, xi = _rays(p, dirs, n, ids, rotate=False)
        L, D = p.n_radial, p.n_dirs
        ball = 4 * math.pi / 3 if p.dim == 3 else math.pi
        E, gc, gk = 0.0, 0.0, torch.zeros_like(Rk)
        e = ((torch.arange(L, device="cuda") + xi[..., None]) / L) ** (1.0 / p.dim)
        for sign in (1.0, -1.0):
            kr = k if sign > 0 else self.anti[k]
            R = Rk.gather(1, kr)
            smax = R + p.dR / 2
            q = ball * smax ** p.dim / (2 * R) ** p.dim / (p.n_rays * L)
            s = smax[..., None] * e
            u = sign * dirs[k]
            I = field.at([c[:, a, None, None] + s * u[..., a, None] for a in range(p.dim)])
            S, Sr, SR = _weights(p, s, R[..., None])
            A = (S * I).sum(2)
            E = E + (q * A).sum(1)
            gc = gc + ((q * -(Sr * I).sum(2))[..., None] * u).sum(1)
            gk.scatter_add_(1, kr, q * ((SR * I).sum(2) - p.dim / R * A))
        f = (eps / 2 * smooth).clamp(max=1.0)[:, None]
        return E, gc, Rk - eps[:, None] / 2 * D * gk - f * (Rk - Rk @ self.mean.T)
