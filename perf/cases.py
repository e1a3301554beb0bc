"""Performance cases of the ray-query library: what its users have it do.

Each case is one call (or one frame, one training step) through the public
entry points of ``paper_2603_00292_amd.api``.  Scenes and rays follow the
recipes of ``paper_2603_00292_amd.workloads`` with their randomness drawn on
the GPU from a seed.  ``listed()`` names twelve cases, ``draw()`` gives others
of the same kinds and ranges.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2603_00292_amd import api, workloads

F64 = torch.float64


def listed():
    return [
        # the smallest call: an editor's pick or a probe batch of 64 rays against a small mesh,
        # all latency and launches
        {"name": "pick", "kind": "closest", "scene": "sphere", "level": 5, "rays": 64},
        # a small batch against a small mesh (the repository's first parity workload)
        {"name": "soup", "kind": "closest", "scene": "soup", "tris": 4096, "rays": 65536},
        # a rendered frame: coherent primary rays and one shadow ray each, 2048 x 2048
        {"name": "camera_frame", "kind": "camera", "level": 8, "width": 2048, "height": 2048},
        # the headline benchmark: 4M incoherent rays at about a million triangles
        {"name": "incoherent", "kind": "closest", "scene": "sphere", "level": 8, "rays": 4194304},
        # incoherent visibility tests, a ragged mid-sized batch
        {"name": "visibility", "kind": "any", "scene": "sphere", "level": 7, "rays": 300007},
        # secondary rays of a two-level scene with instance ids
        {"name": "instanced", "kind": "instanced", "instances": 1024, "rays": 8388608},
        # many meshes with ray batches of uneven sizes, replayed as one HIP graph
        {"name": "batched", "kind": "batched", "meshes": 64, "max_tris": 200000, "max_rays": 300000},
        # query options on a two-level scene: masked and filtered closest hits, and sorted hit lists
        {"name": "filtered_lists", "kind": "lists", "instances": 256, "rays": 250007, "capacity": 8},
        # a differentiable step: forward and backward through the autograd function
        {"name": "train_step", "kind": "train", "nx": 512, "nz": 256, "rays": 1048576},
        # the two-level adjoint with vertex and frame gradients
        {"name": "inst_backward", "kind": "inst_backward", "instances": 1024, "rays": 2000003},
        # ambient occlusion: camera hits, 16 occlusion rays each, resolve
        {"name": "ao", "kind": "ao", "nq": 256, "width": 1024, "height": 1024, "samples": 16},
        # dynamic geometry: a mesh rebuilt on the GPU and traced, and one refitted and traced
        {"name": "dynamic", "kind": "dynamic", "level": 7, "nx": 512, "nz": 256, "rays": 200003},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["closest", "closest", "any", "any", "camera", "instanced", "batched", "lists", "train",
                       "inst_backward", "ao", "dynamic"])
    c = {"kind": kind}
    if kind in ("closest", "any"):
        c["scene"] = rng.choice(["soup", "sphere"])
        if c["scene"] == "soup":
            c["tris"] = _log(rng, 1000, 500000)
        else:
            c["level"] = rng.randint(3, 8)
        c["rays"] = _log(rng, 64, 4194304)
    elif kind == "camera":
        c["level"] = rng.randint(5, 8)
        c["width"], c["height"] = _log(rng, 100, 2048), _log(rng, 100, 2048)
    elif kind == "instanced":
        c["instances"], c["rays"] = _log(rng, 8, 2048), _log(rng, 1000, 8388608)
    elif kind == "batched":
        c["meshes"], c["max_tris"], c["max_rays"] = _log(rng, 4, 64), _log(rng, 5000, 200000), _log(rng, 5000, 300000)
    elif kind == "lists":
        c["instances"], c["rays"], c["capacity"] = _log(rng, 8, 1024), _log(rng, 1000, 500000), rng.randint(1, 16)
    elif kind == "train":
        c["nx"], c["nz"], c["rays"] = _log(rng, 32, 512), _log(rng, 32, 512), _log(rng, 1000, 2097152)
    elif kind == "inst_backward":
        c["instances"], c["rays"] = _log(rng, 8, 2048), _log(rng, 1000, 4194304)
    elif kind == "ao":
        c["nq"], c["width"], c["height"] = _log(rng, 64, 512), _log(rng, 64, 1024), _log(rng, 64, 1024)
        c["samples"] = rng.randint(1, 16)
    else:
        c["level"], c["nx"], c["nz"] = rng.randint(3, 8), _log(rng, 32, 512), _log(rng, 32, 512)
        c["rays"] = _log(rng, 1000, 1000000)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _State:
    """What a program holds before the call; frees its library objects with itself."""

    def __init__(self, **kw):
        self.__dict__.update(kw)

    def __del__(self):
        for k in ("plan", "accel", "accels"):
            v = self.__dict__.get(k)
            for h in (v if isinstance(v, list) else [v]):
                if h is not None:
                    h.close()


@functools.lru_cache(maxsize=None)
def _ctx():
    return api.Context(torch.cuda.current_device())


@functools.lru_cache(maxsize=None)
def _icosphere(level):
    v, f = workloads.icosphere(level)
    return torch.from_numpy(v).cuda(), torch.from_numpy(f.astype(np.int32)).cuda()


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=F64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=F64)


def _unit(x):
    return x / x.norm(dim=1, keepdim=True)


def _rays(o, d, tmin=0.0, tmax=math.inf):
    r = torch.empty((d.shape[0], 8), dtype=F64, device="cuda")
    r[:, 0:3], r[:, 3], r[:, 4:7], r[:, 7] = o, tmin, d, tmax
    return r.float()


def _sphere(g, level):
    v, f = _icosphere(level)
    return (v * (1.0 + 0.04 * (_rand(g, v.shape[0], 1) - 0.5))).float(), f


def _soup(g, n):
    half = 0.025 * math.sqrt(4096.0 / n)
    v = _rand(g, n, 1, 3) + half * (2.0 * _rand(g, n, 3, 3) - 1.0)
    return v.reshape(-1, 3).float(), torch.arange(3 * n, dtype=torch.int32, device="cuda").reshape(n, 3)


def _mesh(case, g):
    """(vertices, indices, half-width and centre of the box of ray origins)"""
    if case["scene"] == "soup":
        return (*_soup(g, case["tris"]), 1.5, 0.5)
    return (*_sphere(g, case["level"]), 1.0, 0.0)


def _box_rays(g, n, half, centre):
    return _rays(centre + half * (2.0 * _rand(g, n, 3) - 1.0), _unit(_randn(g, n, 3)))


def _grid_faces(nx, nz):
    _, f = workloads.grid_mesh(nx, nz, 0.0, 1.0, 0.0, 1.0, np.zeros((nx + 1) * (nz + 1)))
    return torch.from_numpy(f.astype(np.int32)).cuda()


def _grid_vertices(nx, nz, x1, z1, h, x0=0.0, z0=0.0):
    xs = torch.linspace(x0, x1, nx + 1, device="cuda", dtype=F64)
    zs = torch.linspace(z0, z1, nz + 1, device="cuda", dtype=F64)
    X, Z = xs[None, :].expand(nz + 1, -1), zs[:, None].expand(-1, nx + 1)
    return torch.stack([X, h.reshape(nz + 1, nx + 1), Z], -1).reshape(-1, 3).float()


def _down_rays(g, n, nx, nz, y):
    """Rays from the plane y over the grid, within 30 degrees of -y."""
    o = torch.stack([nx * _rand(g, n), y.expand(n), nz * _rand(g, n)], 1)
    ct = 1.0 - (1.0 - math.cos(math.radians(30.0))) * _rand(g, n)
    ph, st = 2 * math.pi * _rand(g, n), torch.sqrt(1.0 - ct * ct)
    return o, torch.stack([st * torch.cos(ph), -ct, st * torch.sin(ph)], 1)


def _pinhole(origin, right, up, width, height):
    o, r, u = (torch.tensor(x, dtype=F64, device="cuda") for x in (origin, right, up))
    fwd = torch.linalg.cross(u, r)
    fwd = fwd / fwd.norm()
    i = torch.arange(width * height, device="cuda")
    x = (2.0 * (i % width).to(F64) / width - 1.0)[:, None]
    y = (1.0 - 2.0 * (i // width).to(F64) / height)[:, None]
    return o, _unit(fwd + x * r + y * u)


def _instances(g, n):
    """Four displaced grids of 10,000 triangles, n scaled, rotated, moved copies."""
    meshes = []
    for s in (0.01, 0.02, 0.05, 0.1):
        v = _grid_vertices(100, 50, 1.0, 0.5, s * _randn(g, 51 * 101), -1.0, -0.5)
        meshes.append((v, _grid_faces(100, 50)))
    side = 20.0 * (n / 1024.0) ** (1.0 / 3.0)
    srt = torch.cat([0.5 + 1.5 * _rand(g, n, 3), _unit(_randn(g, n, 4)), side * (2.0 * _rand(g, n, 3) - 1.0)], 1)
    return meshes, (np.arange(n) % 4).astype(np.uint32), srt.float()


def _quat(q):
    x, y, z, w = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    rows = [1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
            2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
            2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]
    return torch.stack(rows, 1).reshape(-1, 3, 3)


def _surface_points(g, meshes, srt, n):
    """(instance, triangle, world corners (n,3,3), weights (n,3)) of uniform surface points."""
    inst = torch.randint(0, srt.shape[0], (n,), generator=g, device="cuda")
    tri = torch.randint(0, 10000, (n,), generator=g, device="cuda")
    V = torch.stack([v for v, _ in meshes]).to(F64)
    I = torch.stack([f for _, f in meshes]).long()
    s = srt.to(F64)[inst]
    R = _quat(s[:, 3:7])
    p = V[(inst % 4)[:, None], I[inst % 4, tri]] * s[:, None, 0:3]
    w = (R[:, None] * p[:, :, None, :]).sum(-1) + s[:, None, 7:10]
    su, r2 = torch.sqrt(_rand(g, n)), _rand(g, n)
    return inst, tri, w, torch.stack([1 - su, su * (1 - r2), su * r2], 1)


def _secondary(g, meshes, srt, n):
    """Cosine-weighted rays leaving uniform surface points, offset 1e-4."""
    inst, tri, w, b = _surface_points(g, meshes, srt, n)
    p = (b[:, :, None] * w).sum(1)
    nrm = _unit(torch.linalg.cross(w[:, 1] - w[:, 0], w[:, 2] - w[:, 0]))
    nrm = torch.where((nrm * (torch.tensor([0.0, 0.0, 70.0], device="cuda", dtype=F64) - p)).sum(1, keepdim=True) < 0, -nrm, nrm)
    t0 = _unit(w[:, 1] - w[:, 0])
    ph, r = 2 * math.pi * _rand(g, n), torch.sqrt(_rand(g, n))
    d = t0 * (torch.cos(ph) * r)[:, None] + torch.linalg.cross(nrm, t0) * (torch.sin(ph) * r)[:, None] \
        + nrm * torch.sqrt(1 - r * r)[:, None]
    return inst, tri, _rays(p + 1e-4 * nrm, _unit(d))


def _batch_sizes(case):
    """Log-spread triangle and ray counts, in no order (golden-ratio steps)."""
    out = []
    for i in range(case["meshes"]):
        a, b = (i * 0.6180339887498949) % 1.0, (i * 0.4142135623730951 + 0.5) % 1.0
        out.append((round(1000 * (case["max_tris"] / 1000) ** a), round(1000 * (case["max_rays"] / 1000) ** b)))
    return out


def _terrain(g, nq):
    x = torch.linspace(0.0, 16.0, nq + 1, device="cuda", dtype=F64)
    X, Z = x[None, :], x[:, None]
    u = _rand(g, 6, 4).cpu()
    h = torch.zeros((nq + 1, nq + 1), device="cuda", dtype=F64)
    for a, f, th, ph in u.tolist():
        th, f = 2 * math.pi * th, 1.0 + 3.0 * f
        h += (0.2 + 0.4 * a) * torch.sin(f * (X * math.cos(th) + Z * math.sin(th)) + 2 * math.pi * ph)
    return _grid_vertices(nq, nq, 16.0, 16.0, h), _grid_faces(nq, nq)


def prepare(case, seed):
    kind, g, ctx = case["kind"], _gen(seed), _ctx()
    S = _State(kind=kind)
    if kind in ("closest", "any"):
        v, f, half, centre = _mesh(case, g)
        S.rays = _box_rays(g, case["rays"], half, centre)
        S.accel = api.Accel(ctx, [(v, f)])
    elif kind == "camera":
        v, f = _sphere(g, case["level"])
        th = math.tan(math.radians(20.0))
        o, d = _pinhole((0.0, 0.0, 3.0), (th * case["width"] / case["height"], 0.0, 0.0), (0.0, th, 0.0),
                        case["width"], case["height"])
        S.rays = _rays(o, d)
        # shadow rays from the sphere just outside the mesh toward the light
        b = (d * o).sum(1)
        disc = b * b - ((o * o).sum() - 1.0201 ** 2)
        p = o + torch.where(disc >= 0, -b - torch.sqrt(disc.clamp(min=0)), 3.0)[:, None] * d
        to = torch.tensor([2.0, 2.0, 2.0], device="cuda", dtype=F64) - p
        dist = to.norm(dim=1)
        S.shadow = _rays(p, to / dist[:, None], 0.0, dist)
        S.accel = api.Accel(ctx, [(v, f)])
    elif kind in ("instanced", "lists"):
        meshes, im, srt = _instances(g, case["instances"])
        inst, tri, S.rays = _secondary(g, meshes, srt, case["rays"])
        S.accel = api.Accel(ctx, meshes, im, srt.cpu().numpy())
        if kind == "lists":
            S.capacity = case["capacity"]
            S.skip_inst, S.skip_prim = inst.int(), tri.int()
            S.ray_masks = torch.randint(1, 16, (case["rays"],), generator=g, device="cuda", dtype=torch.int32)
            S.accel.set_instance_masks(1 << (np.arange(case["instances"]) % 4))
    elif kind == "batched":
        sizes = _batch_sizes(case)
        S.accels, rays = [], []
        for nt, nr in sizes:
            S.accels.append(api.Accel(ctx, [_soup(g, nt)], device_build=True))
            rays.append(_box_rays(g, nr, 1.5, 0.5))
        S.hits = torch.empty((sum(nr for _, nr in sizes), 4), dtype=torch.float32, device="cuda")
        S.plan = api.BatchPlan(ctx, S.accels, rays, list(S.hits.split([nr for _, nr in sizes])))
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        S.graph = S.plan.graph_exec(side)
    elif kind == "train":
        nx, nz = case["nx"], case["nz"]
        v = _grid_vertices(nx, nz, nx, nz, 0.05 * _randn(g, (nx + 1) * (nz + 1)))
        o, d = _down_rays(g, case["rays"], nx, nz, v[:, 1].max().to(F64))
        S.accel = api.Accel(ctx, [(v, _grid_faces(nx, nz))])
        S.inputs = [x.float().contiguous().requires_grad_() for x in (v, o, d)]
        S.grads = [_randn(g, case["rays"]).float() for _ in range(3)]
    elif kind == "inst_backward":
        meshes, im, srt = _instances(g, case["instances"])
        inst, tri, w, b = _surface_points(g, meshes, srt, case["rays"])
        d = _unit(_randn(g, case["rays"], 3))
        S.rays = _rays((b[:, :, None] * w).sum(1) - d * (0.5 + 10.0 * _rand(g, case["rays"], 1)), d)
        # the adjoint reads a hit's triangle id; its t, u, v are formed anew
        S.hits = torch.zeros((case["rays"], 4), dtype=torch.float32, device="cuda")
        S.hits.view(torch.int32)[:, 1] = tri.int()
        S.inst = inst.int()
        S.d_tuv = _randn(g, case["rays"], 3).float()
        S.meshes, S.srt = meshes, srt
        S.accel = api.Accel(ctx, meshes, im, srt.cpu().numpy())
    elif kind == "ao":
        v, f = _terrain(g, case["nq"])
        fwd = np.array([0.0, -6.0, 11.0]) / math.sqrt(157.0)
        right = np.cross(fwd, [0.0, 1.0, 0.0])
        right /= np.linalg.norm(right)
        half = math.tan(math.radians(30.0))
        up = np.cross(right, fwd) * half
        right = right * half * case["width"] / case["height"]
        S.rays = _rays(*_pinhole((8.0, 6.0, -2.0), right.tolist(), up.tolist(), case["width"], case["height"]))
        S.xi = torch.rand((S.rays.shape[0], case["samples"], 2), generator=g, device="cuda")
        S.accel = api.Accel(ctx, [(v, f)])
    else:
        S.mesh = _sphere(g, case["level"])
        S.mesh_rays = _box_rays(g, case["rays"], 1.0, 0.0)
        nx, nz = case["nx"], case["nz"]
        h = 0.05 * _randn(g, 2, (nx + 1) * (nz + 1))
        S.moved = _grid_vertices(nx, nz, nx, nz, h[1])
        S.rays = _rays(*_down_rays(g, case["rays"], nx, nz, S.moved[:, 1].max().to(F64)))
        S.accel = api.Accel(ctx, [(_grid_vertices(nx, nz, nx, nz, h[0]), _grid_faces(nx, nz))])
    return S


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _tuv(hits):
    """The three parts of hit records: t, triangle ids, (u, v)."""
    return hits[..., 0], hits.view(torch.int32)[..., 1], hits[..., 2:]


def run(S):
    if S.kind == "closest":
        return _tuv(api.trace_closest(S.accel, S.rays)[0])
    if S.kind == "any":
        return api.trace_any(S.accel, S.rays)
    if S.kind == "camera":
        hits, _ = api.trace_closest(S.accel, S.rays)
        return *_tuv(hits), api.trace_any(S.accel, S.shadow)
    if S.kind == "instanced":
        hits, inst = api.trace_closest(S.accel, S.rays, want_inst=True)
        return *_tuv(hits), inst
    if S.kind == "batched":
        api.graph_launch(S.graph)
        return _tuv(S.hits)
    if S.kind == "lists":
        kw = {"ray_masks": S.ray_masks, "skip_inst": S.skip_inst, "skip_prim": S.skip_prim, "want_inst": True}
        near, near_inst = api.trace_closest_ex(S.accel, S.rays, **kw)
        hits, inst, counts = api.trace_all(S.accel, S.rays, S.capacity, **kw)
        return *_tuv(near), near_inst, *_tuv(hits), inst, counts
    if S.kind == "train":
        v, o, d = S.inputs
        t, u, w, prim = api.RayQueryFn.apply(S.accel, v, o, d, 0.0, math.inf)
        return t.detach(), u.detach(), w.detach(), prim, *torch.autograd.grad([t, u, w], S.inputs, S.grads)
    if S.kind == "inst_backward":
        dv = torch.zeros((sum(S.accel.vertex_counts), 3), dtype=torch.float32, device="cuda")
        ds = torch.zeros((S.accel.instance_count, 10), dtype=torch.float32, device="cuda")
        do, dd = api.trace_backward_instances(S.accel, S.rays, S.hits, S.inst, S.d_tuv, dv, ds)
        return do, dd, dv, ds
    if S.kind == "ao":
        ao, hits, rays, occ = api.ambient_occlusion(S.accel, S.rays, S.xi, 1e-4, 1.0)
        return ao, *_tuv(hits), rays, occ
    rebuilt = api.Accel(_ctx(), [S.mesh], device_build=True)
    a, _ = api.trace_closest(rebuilt, S.mesh_rays)
    rebuilt.close()
    S.accel.refit(S.moved)
    b, _ = api.trace_closest(S.accel, S.rays)
    return *_tuv(a), *_tuv(b)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _query_work(rays, tris, out):
    """One query: rays read, `out` bytes a ray written, and the geometry (36
    bytes a triangle, at most one triangle a ray) read; a descent of a 4-wide
    tree over the triangles (24 flops a box) and one triangle test (60)."""
    depth = max(1.0, math.log(max(tris, 4), 4))
    return rays * (32 + out) + 36 * min(rays, tris), rays * (depth * 4 * 24 + 60)


def work(case):
    k = case["kind"]
    sphere = 20 * 4 ** case["level"] if "level" in case else 0
    n = case.get("rays", 0)
    if k in ("closest", "any"):
        b, f = _query_work(n, sphere if case["scene"] == "sphere" else case["tris"], 16 if k == "closest" else 1)
    elif k == "camera":
        n = case["width"] * case["height"]
        b, f = (x + y for x, y in zip(_query_work(n, sphere, 16), _query_work(n, sphere, 1)))
    elif k == "instanced":
        b, f = _query_work(n, 40000, 20)
    elif k == "lists":
        b, f = (x + y for x, y in zip(_query_work(n, 40000, 20 + 12), _query_work(n, 40000, 20 * case["capacity"] + 4)))
    elif k == "batched":
        parts = [_query_work(nr, nt, 16) for nt, nr in _batch_sizes(case)]
        b, f = sum(p[0] for p in parts), sum(p[1] for p in parts)
    elif k == "train":
        t = 2 * case["nx"] * case["nz"]
        b, f = _query_work(n, t, 16)
        # backward: rays, gradients of (t, u, v), ids, triangles read; ray and vertex gradients written
        b, f = b + n * (32 + 12 + 4 + 24) + 48 * t + 6 * t, f + 200 * n
    elif k == "inst_backward":
        b, f = n * (32 + 12 + 4 + 4 + 24) + 40000 * 48 + 20604 * 12 + case["instances"] * 176, 400 * n
    elif k == "ao":
        p, t = case["width"] * case["height"], 2 * case["nq"] ** 2
        (b0, f0), (b1, f1) = _query_work(p, t, 16), _query_work(p * case["samples"], t, 1)
        b, f = b0 + b1 + p * (case["samples"] * (8 + 32 + 1) + 4), f0 + f1 + 120 * p * case["samples"]
    else:
        t = 2 * case["nx"] * case["nz"]
        (b0, f0), (b1, f1) = _query_work(n, sphere, 16), _query_work(n, t, 16)
        # build: triangles read, records and boxes written; refit the same
        b, f = b0 + b1 + sphere * (18 + 48 + 32) + t * (18 + 48 + 32), f0 + f1 + 60 * (sphere + t)
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same results in 64 bits (plain torch)
# ---------------------------------------------------------------------------
def _hit64(o, d, tri):
    """(t, u, v) of o + t d = (1-u-v) v0 + u v1 + v v2; t = inf outside the triangle or behind."""
    e1, e2, s = tri[..., 1, :] - tri[..., 0, :], tri[..., 2, :] - tri[..., 0, :], o - tri[..., 0, :]
    p, q = torch.linalg.cross(d, e2), torch.linalg.cross(s, e1)
    det = (e1 * p).sum(-1)
    t, u, v = (e2 * q).sum(-1) / det, (s * p).sum(-1) / det, (d * q).sum(-1) / det
    ok = (det != 0) & (u >= 0) & (v >= 0) & (u + v <= 1) & (t >= 0)
    return torch.where(ok, t, math.inf), u, v


def _nearest(o, d, tris):
    """Nearest of the candidate triangles (n, c, 3, 3), or of all (1, c, 3, 3): (t, index, u, v)."""
    t, u, v = _hit64(o[:, None].expand(-1, tris.shape[1], -1), d[:, None].expand(-1, tris.shape[1], -1),
                     tris.expand(o.shape[0], -1, -1, -1))
    t, i = t.min(1)
    hit = torch.isfinite(t)
    u, v = (torch.where(hit, x.gather(1, i[:, None])[:, 0], 0.0) for x in (u, v))
    return t, i, u, v


def _brute(rays, v, f, chunk=1 << 23):
    tris, r = v.to(F64)[f.long()][None], rays.to(F64)
    step = max(1, chunk // f.shape[0])
    parts = [_nearest(x[:, 0:3], x[:, 4:7], tris) for x in r.split(step)]
    return [torch.cat(x) for x in zip(*parts)]


def _grid_hits(o, d, v, f, nx, nz):
    """Nearest hits of steep rays on a displaced grid of unit quads: the 3 x 3
    quads about the crossing of y = 0 hold them all (heights well under 1/2,
    rays within 30 degrees of vertical).  Returns (t, triangle, u, v)."""
    tris = v[f.long()]
    out = []
    for oo, dd in zip(o.split(1 << 18), d.split(1 << 18)):
        x = oo - dd * (oo[:, 1] / dd[:, 1])[:, None]
        i, j = x[:, 0].floor().long(), x[:, 2].floor().long()
        k = torch.arange(9, device="cuda")
        ii, jj = i[:, None] + k % 3 - 1, j[:, None] + k // 3 - 1
        inside = (ii >= 0) & (ii < nx) & (jj >= 0) & (jj < nz)
        quad = jj.clamp(0, nz - 1) * nx + ii.clamp(0, nx - 1)
        cand = torch.cat([2 * quad, 2 * quad + 1], 1)
        c = torch.where(torch.cat([inside, inside], 1)[..., None, None], tris[cand], 0.0)
        t, w, a, b = _nearest(oo, dd, c)
        out.append((t, cand.gather(1, w[:, None])[:, 0], a, b))
    return [torch.cat(y) for y in zip(*out)]


def _adjoint(o, d, tri, g):
    """(t, weights, lambda = M^-T g) of M = [-d | v1 - v0 | v2 - v0]."""
    e1, e2, s = tri[:, 1] - tri[:, 0], tri[:, 2] - tri[:, 0], o - tri[:, 0]
    r0, r1, r2 = torch.linalg.cross(e1, e2), torch.linalg.cross(d, e2), torch.linalg.cross(e1, d)
    det = -(d * r0).sum(1)
    r0, r1, r2 = (r / det[:, None] for r in (r0, r1, r2))
    t, u, v = (r0 * s).sum(1), (r1 * s).sum(1), (r2 * s).sum(1)
    lam = g[:, 0:1] * r0 + g[:, 1:2] * r1 + g[:, 2:3] * r2
    return t, torch.stack([1 - u - v, u, v], 1), lam


def exact(case, seed):
    k = case["kind"]
    if k == "closest":
        g = _gen(seed)
        v, f, half, centre = _mesh(case, g)
        if f.shape[0] * case["rays"] > 3e8:
            return None
        rays = _box_rays(g, case["rays"], half, centre)
        t, _, a, b = _brute(rays, v, f)
        return t, None, torch.stack([a, b], 1)
    if k == "train":
        S = prepare(case, seed)
        v, o, d = (x.detach().to(F64) for x in S.inputs)
        f = _grid_faces(case["nx"], case["nz"])
        t, prim, a, b = _grid_hits(o, d, v, f, case["nx"], case["nz"])
        hit = torch.isfinite(t)
        gr = torch.stack(S.grads, 1).to(F64)
        tt, w, lam = _adjoint(o[hit], d[hit], v[f.long()[prim[hit]]], gr[hit])
        do, dd = torch.zeros_like(o), torch.zeros_like(d)
        do[hit], dd[hit] = lam, tt[:, None] * lam
        dv = torch.zeros_like(v)
        for c in range(3):
            dv.index_add_(0, f.long()[prim[hit], c], -w[:, c:c + 1] * lam)
        return t, a, b, None, dv, do, dd
    if k == "inst_backward":
        S = prepare(case, seed)
        s, inst, tri = S.srt.to(F64), S.inst.long(), S.hits.view(torch.int32)[:, 1].long()
        V = torch.stack([v for v, _ in S.meshes]).to(F64)
        I = torch.stack([f for _, f in S.meshes]).long()
        ids = I[inst % 4, tri]
        obj = V[(inst % 4)[:, None], ids]
        R = _quat(s[:, 3:7])[inst]
        scaled = obj * s[inst][:, None, 0:3]
        tri_w = (R[:, None] * scaled[:, :, None, :]).sum(-1) + s[inst][:, None, 7:10]
        r = S.rays.to(F64)
        t, w, lam = _adjoint(r[:, 0:3], r[:, 4:7], tri_w, S.d_tuv.to(F64))
        # object vertices: -w_k S R^T lambda; frames: the chain rule through T + R(q/|q|)(S p)
        rl = (R * lam[:, :, None]).sum(1)
        dv = torch.zeros((4 * 5151, 3), device="cuda", dtype=F64)
        for c in range(3):
            dv.index_add_(0, (inst % 4) * 5151 + ids[:, c], -w[:, c:c + 1] * s[inst, 0:3] * rl)
        p = (w[:, :, None] * obj).sum(1)
        a = p * s[inst, 0:3]
        q = s[inst, 3:7]
        qn = q.norm(dim=1, keepdim=True)
        x, y, z, qw = (q / qn).unbind(1)
        m = -lam[:, :, None] * a[:, None, :]   # dL/dR
        gx = 2 * (y * (m[:, 0, 1] + m[:, 1, 0]) + z * (m[:, 0, 2] + m[:, 2, 0]) - 2 * x * (m[:, 1, 1] + m[:, 2, 2]) + qw * (m[:, 2, 1] - m[:, 1, 2]))
        gy = 2 * (x * (m[:, 0, 1] + m[:, 1, 0]) + z * (m[:, 1, 2] + m[:, 2, 1]) - 2 * y * (m[:, 0, 0] + m[:, 2, 2]) + qw * (m[:, 0, 2] - m[:, 2, 0]))
        gz = 2 * (x * (m[:, 0, 2] + m[:, 2, 0]) + y * (m[:, 1, 2] + m[:, 2, 1]) - 2 * z * (m[:, 0, 0] + m[:, 1, 1]) + qw * (m[:, 1, 0] - m[:, 0, 1]))
        gw = 2 * (x * (m[:, 2, 1] - m[:, 1, 2]) + y * (m[:, 0, 2] - m[:, 2, 0]) + z * (m[:, 1, 0] - m[:, 0, 1]))
        gq, qh = torch.stack([gx, gy, gz, gw], 1), q / qn
        gq = (gq - qh * (qh * gq).sum(1, keepdim=True)) / qn
        ds = torch.zeros((s.shape[0], 10), device="cuda", dtype=F64)
        ds.index_add_(0, inst, torch.cat([-rl * p, gq, -lam], 1))
        return lam, t[:, None] * lam, dv, ds
    if k == "dynamic":
        S = prepare(case, seed)
        r = S.rays.to(F64)
        t, _, a, b = _grid_hits(r[:, 0:3], r[:, 4:7], S.moved.to(F64), _grid_faces(case["nx"], case["nz"]), case["nx"], case["nz"])
        return None, None, None, t, None, torch.stack([a, b], 1)
    return None
