"""Timed cases of the library: the queries, updates and builds that a program
using it makes, at sizes from its own workloads, tests and benchmark.

A case is a scene (the unit room with boxes and icospheres of
workloads.make_scene), a distance-field grid, and one call or one short
sequence of calls.  Scenes, trees and grids of the trace cases are kept for the
process, as a program keeps its resident scene from frame to frame; every state
is a new frame of it: another camera position, other ray directions.
"""
import functools
import math

import numpy as np
import torch

import paper_2305_07253_amd as hyb
from paper_2305_07253_amd import workloads
from paper_2305_07253_amd.autograd import df_hit

FORMATS = {"f32": hyb.SDF_F32, "f16": hyb.SDF_F16, "i8": hyb.SDF_I8_BRICK}
F64 = torch.float64


def _case(name, kind, **options):
    """detail: 6 for the finely tessellated objects of the GI-shaped scene, 1
    for those of the tiny room; rays: 0 for all of width x height x spp."""
    case = dict(kind=kind, scene=2, objects=500, detail=6, n=128, fmt="f32", tau=0.0, tmax=0.5,
                width=1920, height=1080, spp=1, rays=0)
    case.update(options)
    return dict(case, name=name) if name else case


def listed():
    return [
        # a handful of probe rays against a small scene: launch latency
        _case("probe rays, small scene", "trace", scene=1, objects=30, detail=1, n=32, tau=1.0, tmax=2.0,
              width=40, height=25),
        # one diffuse bounce of a full-screen pass, one ray a pixel, switching at
        # the start of the ray (the benchmark's query) and after one voxel
        _case("gi 1080p threshold 0", "trace"),
        _case("gi 1080p threshold 1", "trace", tau=1.0),
        # the exact reference that programs compare with, half resolution
        _case("triangles only 960x540", "bvh", width=960, height=540),
        # shadow rays to an area light, triangles at both ends
        _case("shadow rays 720p", "shadow", tau=1.0, width=1280, height=720),
        # short occlusion rays through half-precision samples, ragged ray count
        _case("ambient occlusion f16", "trace", fmt="f16", n=97, tau=1.0, tmax=0.1, rays=1234567),
        # a detailed scene, fine grid in its smallest storage, several rays a pixel
        _case("fine grid i8, 4 rays a pixel", "trace", scene=3, objects=5000, n=256, fmt="i8", tau=1.0, spp=4,
              width=1280, height=720),
        # many scenes of uneven size served by one launch
        _case("12 scenes in one launch", "batch", scene=4, objects=12, tau=1.0),
        # one step of fitting a grid by gradient descent: update, forward, backward
        _case("refit step 128^3", "refit", width=1024, height=1024),
        # a field that changes every frame: new samples, then the frame's rays
        _case("new samples and 360p rays f16", "update", fmt="f16", n=96, width=640, height=360),
        # distance field of a loaded mesh, at the resolution the queries use
        _case("distance field of a mesh 128^3", "build"),
        # a small scene loaded from scratch: tree and distance field
        _case("load a small scene", "load", scene=1, objects=30, detail=1, n=32),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["trace", "trace", "trace", "bvh", "shadow", "batch", "refit", "update", "build", "load"])
    objects, detail = log(20, 700), rng.choice([1, 6, 6])
    options = dict(scene=rng.randrange(5, 100), objects=objects, detail=detail, n=log(24, 150),
                   fmt=rng.choice(list(FORMATS)), tau=rng.choice([0.0, 0.5, 1.0, 2.0, 4.0]),
                   tmax=round(rng.uniform(0.05, 1.0), 3))
    rays = log(500, 2000000)
    options["width"] = max(8, int(math.sqrt(rays * 16 / 9)))
    options["height"] = rays // options["width"] + 1
    options["rays"] = rays
    if kind == "refit":
        options.update(fmt="f32", tau=0.0)
    elif kind in ("update", "bvh"):
        options.update(tau=0.0)
    elif kind == "batch":
        options.update(objects=rng.randrange(2, 13), n=128, width=0, height=0, rays=0, fmt="f32")
    elif kind in ("build", "load"):
        options.update(objects=min(objects, 500 if kind == "build" else 60), n=log(24, 128), tau=0.0, tmax=0.5,
                       width=0, height=0, rays=0)
    return _case(None, kind, **options)


# ----------------------------------------------------------------------------
# scenes, grids and rays
# ----------------------------------------------------------------------------


@functools.lru_cache(maxsize=None)
def _scene(seed, objects, detail):
    size = min(0.25, 0.06 * (500.0 / objects) ** (1.0 / 3.0))
    kinds = None
    if detail == 1:  # two boxes to every icosphere, as in the tiny room
        kinds = np.where(np.arange(objects) * 3 < objects * 2, workloads.KIND_BOX, workloads.KIND_ICO)
    return workloads.make_scene(seed, objects, size / 10.0, size, box_subdiv=detail, ico_splits=2 if detail > 1 else 1,
                                kinds=kinds)


@functools.lru_cache(maxsize=None)
def _bvh(seed, objects, detail):
    scene = _scene(seed, objects, detail)
    return hyb.build_bvh(scene.verts, scene.tris)


@functools.lru_cache(maxsize=None)
def _sdf(seed, objects, detail, n, fmt):
    return hyb.build_sdf(_bvh(seed, objects, detail), n, workloads.room_grid(n), fmt=FORMATS[fmt])


@functools.lru_cache(maxsize=None)
def _mesh(seed, objects, detail):
    """Corner positions of every triangle on the GPU, (T, 3, 3) in 64 bits."""
    return torch.from_numpy(_scene(seed, objects, detail).triangle_soup()).cuda().double()


def _hit_triangles(o, d, tri):
    """t, u, v of rays against triangles in 64 bits; t is inf for a miss."""
    e1, e2 = tri[..., 1, :] - tri[..., 0, :], tri[..., 2, :] - tri[..., 0, :]
    p = torch.linalg.cross(d, e2, dim=-1)
    det = (e1 * p).sum(-1)
    s = o - tri[..., 0, :]
    q = torch.linalg.cross(s, e1, dim=-1)
    u, v, t = (s * p).sum(-1) / det, (d * q).sum(-1) / det, (e2 * q).sum(-1) / det
    hit = (det != 0) & (u >= 0) & (v >= 0) & (u + v <= 1) & (t > 0)
    return torch.where(hit, t, math.inf), u, v


def _gbuffer(scene_key, width, height, gen):
    """Visible point and normal of every pixel of a camera near the workloads'
    one, in 8x8-tile order: (n, 3) each, in 64 bits."""
    tri = _mesh(*scene_key)
    moved = (torch.rand(3, generator=gen, dtype=F64) - 0.5) * 0.04
    eye = torch.from_numpy(workloads.CAMERA_EYE).double() + moved * torch.tensor([1.0, 1.0, 0.5], dtype=F64)
    right, up, fwd = (torch.from_numpy(np.ascontiguousarray(x)).double().cuda() for x in workloads._camera_basis())
    eye = eye.cuda()
    f = height / 2.0 / math.tan(math.radians(workloads.CAMERA_VFOV_DEG) / 2.0)

    def direction(pixel):
        x, y = (pixel % width + 0.5 - width / 2.0) / f, (height / 2.0 - pixel // width - 0.5) / f
        return fwd + x[:, None] * right + y[:, None] * up

    pixel = torch.arange(width * height, device="cuda")
    nearest = torch.full((width * height,), 1 << 62, device="cuda")

    def keep(pixels, ids):
        t = _hit_triangles(eye, direction(pixels), tri[ids])[0]
        key = torch.where(t < 8, (t.clamp(max=8) * (1 << 30)).long() << 26 | ids, 1 << 62)
        nearest.scatter_reduce_(0, pixels, key, "amin")

    for k in range(12):  # the room's walls: every pixel
        keep(pixel, torch.full_like(pixel, k))
    local = tri - eye
    z = (local @ fwd).clamp(min=1e-9)
    x, y = (local @ right) / z * f + width / 2.0 - 0.5, height / 2.0 - (local @ up) / z * f - 0.5
    x0, x1 = x.amin(1).ceil().clamp(0, width).long(), x.amax(1).floor().clamp(-1, width - 1).long()
    y0, y1 = y.amin(1).ceil().clamp(0, height).long(), y.amax(1).floor().clamp(-1, height - 1).long()
    facing = (torch.linalg.cross(tri[:, 1] - tri[:, 0], tri[:, 2] - tri[:, 0], dim=-1) * (tri[:, 0] - eye)).sum(1) < 0
    seen = facing & (z.amin(1) > 0.01) & (x1 >= x0) & (y1 >= y0)
    seen[:12] = False
    seen = seen.nonzero()[:, 0]
    for ids in seen.split(1 << 16):
        w = x1[ids] - x0[ids] + 1
        count = w * (y1[ids] - y0[ids] + 1)
        which = torch.repeat_interleave(torch.arange(len(ids), device="cuda"), count)
        k = torch.arange(len(which), device="cuda") - (count.cumsum(0) - count)[which]
        ids, w = ids[which], w[which]
        keep((y0[ids] + k // w) * width + x0[ids] + k % w, ids)
    ids = (nearest & ((1 << 26) - 1)).clamp(max=len(tri) - 1)
    d = direction(pixel)
    t = ((nearest >> 26).double() / (1 << 30)).clamp(max=8)
    normal = torch.linalg.cross(tri[ids, 1] - tri[ids, 0], tri[ids, 2] - tri[ids, 0], dim=-1)
    normal = normal / normal.norm(dim=1, keepdim=True)
    normal = torch.where(((d * normal).sum(1) > 0)[:, None], -normal, normal)
    # depth from the plane of the triangle seen, not from the sorting key
    plane = (normal * (tri[ids, 0] - eye)).sum(1) / (normal * d).sum(1)
    t = torch.where((plane - t).abs() < 1e-6, plane, t)
    px, py = pixel % width, pixel // width
    order = (((py // 8 * ((width + 7) // 8) + px // 8) * 8 + py % 8) * 8 + px % 8).argsort()
    return (eye + t[:, None] * d)[order], normal[order]


def _rays(case, scene_key, width, height, gen, spp=1, rays=0, bias=1e-5):
    """(6, n) rays leaving the visible points along cosine-weighted directions,
    or, for shadow rays, toward an area light with their lengths."""
    p, normal = _gbuffer(scene_key, width, height, gen)
    p, normal = p.repeat_interleave(spp, 0), normal.repeat_interleave(spp, 0)
    gpu = torch.Generator("cuda").manual_seed(int(torch.randint(1 << 40, (1,), generator=gen)))
    o = (p + bias * normal).float()
    length = None
    if case["kind"] == "shadow":
        light = torch.rand(len(p), 3, generator=gpu, device="cuda", dtype=F64)
        light = light * torch.tensor([0.3, 0.0, 0.3], device="cuda", dtype=F64)
        light = light + torch.tensor([0.35, 0.999, 0.35], device="cuda", dtype=F64)
        d = light - o
        length = d.norm(dim=1).float()
    else:
        s = torch.randn(len(p), 3, generator=gpu, device="cuda", dtype=F64)
        d = normal + s / s.norm(dim=1, keepdim=True)
    d = (d / d.norm(dim=1, keepdim=True)).float()
    both = torch.cat([o, d], 1)[: rays or None]
    return both.T.contiguous(), None if length is None else length[: rays or None].contiguous()


@functools.lru_cache(maxsize=8)
def _field(seed, objects, detail, n):
    """Samples of the scene's own distance field from its primitives, (n^3,) in
    64 bits: what a program that models a field without a mesh hands over."""
    scene, grid4 = _scene(seed, objects, detail), workloads.room_grid(n).astype(np.float64)
    axis = torch.arange(n, device="cuda", dtype=F64) * grid4[3] + grid4[0]
    p = torch.stack(torch.meshgrid(axis, axis, axis, indexing="ij"), -1).flip(-1).reshape(-1, 3)
    out = (0.5 - (p - 0.5).abs()).amin(1)
    for g in range(1, len(scene.group_kind)):
        c, rot, ext = (torch.from_numpy(np.asarray(x[g])).double().cuda()
                       for x in (scene.centers, scene.rots, scene.extents))
        q = p - c
        if scene.group_kind[g] == workloads.KIND_BOX:
            q = (q @ rot).abs() - ext
            dist = q.clamp(min=0).norm(dim=1) + q.amax(1).clamp(max=0)
        else:
            dist = q.norm(dim=1) - ext[0]
        out = torch.minimum(out, dist)
    return out


def _samples(case, gen):
    """Samples of a field in motion: the scene's own, off by a small part of a voxel."""
    field = _field(case["scene"], case["objects"], case["detail"], case["n"])
    gpu = torch.Generator("cuda").manual_seed(int(torch.randint(1 << 40, (1,), generator=gen)))
    h = float(workloads.room_grid(case["n"])[3])
    return (field + 0.02 * h * torch.randn(len(field), generator=gpu, device="cuda", dtype=F64)).float()


# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------


def _key(case):
    return case["scene"], case["objects"], case["detail"]


def prepare(case, seed):
    gen = torch.Generator().manual_seed(int(seed))
    state = dict(case=case, kind=case["kind"])
    frame = dict(width=case["width"], height=case["height"], spp=case["spp"], rays=case["rays"])
    if case["kind"] in ("trace", "bvh", "shadow"):
        state["bvh"] = _bvh(*_key(case))
        if case["kind"] != "bvh":
            state["sdf"] = _sdf(*_key(case), case["n"], case["fmt"])
        state["rays"], state["length"] = _rays(case, _key(case), gen=gen, **frame)
    elif case["kind"] == "batch":
        items = []
        for spec in workloads.batch_specs(case["scene"], case["objects"], tris=(1e3, 2e5), rays=(1e3, 1e6)):
            key = (spec.seed, spec.n_objects, 6)
            items.append(dict(bvh=_bvh(*key), sdf=_sdf(*key, spec.n_grid, case["fmt"]), tmax=case["tmax"],
                              rays=_rays(case, key, spec.width, spec.height, gen)[0], threshold=case["tau"]))
        state["batch"] = hyb.Batch(items)
    elif case["kind"] in ("refit", "update"):
        grid4 = workloads.room_grid(case["n"])
        state.update(grid4=grid4, values=_samples(case, gen))
        state["rays"] = _rays(case, _key(case), gen=gen, bias=float(grid4[3]), **frame)[0]
        state["sdf"] = hyb.sdf_from_grid(state["values"], grid4, fmt=FORMATS[case["fmt"]])
        if case["kind"] == "refit":
            state["theta"] = state["values"].requires_grad_()
            state["grad_t"] = torch.randn(state["rays"].shape[1], generator=torch.Generator("cuda").manual_seed(
                int(seed) + 1), device="cuda")
    else:
        # another placement of the same scene in its grid for every seed
        scene = _scene(*_key(case))
        moved = (torch.rand(3, generator=gen).numpy() - 0.5).astype(np.float32) * np.float32(0.01)
        state.update(verts=scene.verts + moved, tris=scene.tris, grid4=workloads.room_grid(case["n"]))
        if case["kind"] == "build":
            state["bvh"] = hyb.build_bvh(state["verts"], state["tris"])
    return state


def run(state):
    case, kind = state["case"], state["kind"]
    if kind == "trace":
        return hyb.trace(state["bvh"], state["sdf"], state["rays"], case["tmax"], case["tau"])
    if kind == "bvh":
        return hyb.trace_bvh(state["bvh"], state["rays"], case["tmax"])
    if kind == "shadow":
        return hyb.trace_shadow(state["bvh"], state["sdf"], state["rays"], 2.0, case["tau"], case["tau"],
                                tmax_ray=state["length"])
    if kind == "batch":
        return state["batch"].launch()
    if kind == "refit":
        theta = state["theta"]
        theta.grad = None
        t = df_hit(theta, state["grid4"], state["rays"], case["tmax"], sdf=state["sdf"])
        t.backward(state["grad_t"])
        return t.detach(), theta.grad
    if kind == "update":
        hyb.sdf_update(state["sdf"], state["values"])
        return hyb.trace_df(state["sdf"], state["rays"], case["tmax"])
    bvh = state["bvh"] if kind == "build" else hyb.build_bvh(state["verts"], state["tris"])
    return hyb.sdf_read(hyb.build_sdf(bvh, case["n"], state["grid4"], fmt=FORMATS[case["fmt"]]))


def work(case):
    """Bytes of one pass: rays in and hits out, the samples and the triangles once."""
    sample = {"f32": 4, "f16": 2, "i8": 1}[case["fmt"]]
    rays = case["rays"] or case["width"] * case["height"] * case["spp"]
    if case["kind"] == "batch":
        total = 0
        for spec in workloads.batch_specs(case["scene"], case["objects"], tris=(1e3, 2e5), rays=(1e3, 1e6)):
            total += 40 * spec.n_rays + sample * spec.n_grid ** 3 + 36 * _scene(spec.seed, spec.n_objects, 6).n_tris
        return dict(bytes=total, flops=0)
    nodes, mesh = case["n"] ** 3, 36 * _scene(*_key(case)).n_tris
    if case["kind"] in ("build", "load"):
        return dict(bytes=mesh + 4 * nodes, flops=0)
    if case["kind"] == "refit":  # samples and their gradient, t out, t and its gradient in
        return dict(bytes=8 * nodes + 36 * rays, flops=0)
    if case["kind"] == "update":
        return dict(bytes=4 * nodes + 40 * rays, flops=0)
    extra = {"trace": sample * nodes, "bvh": 0, "shadow": sample * nodes + 4 * rays}[case["kind"]]
    return dict(bytes=40 * rays + mesh + extra, flops=0)


# ----------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------


def _mesh_distance(tri, p, inside):
    """Signed distance of points to a mesh, brute force: nearest triangle, and
    solid where the winding number plus `inside` is at least 1."""
    best = torch.full((len(p),), math.inf, device="cuda", dtype=F64)
    angle = torch.zeros_like(best)
    for a, b, c in tri:
        n = torch.linalg.cross(b - a, c - a)
        face = torch.ones(len(p), dtype=torch.bool, device="cuda")
        for s, e in ((a, b), (b, c), (c, a)):
            w, edge = p - s, e - s
            k = ((w @ edge) / (edge @ edge)).clamp(0, 1)
            best = torch.minimum(best, (w - k[:, None] * edge).square().sum(1))
            face &= w @ torch.linalg.cross(n, edge) >= 0
        plane = ((p - a) @ n).square() / (n @ n)
        best = torch.where(face, torch.minimum(best, plane), best)
        x, y, z = a - p, b - p, c - p
        lx, ly, lz = x.norm(dim=1), y.norm(dim=1), z.norm(dim=1)
        num = (x * torch.linalg.cross(y, z)).sum(1)
        den = lx * ly * lz + (x * y).sum(1) * lz + (y * z).sum(1) * lx + (z * x).sum(1) * ly
        angle += 2 * torch.atan2(num, den)
    solid = (angle / (4 * math.pi)).round() + inside >= 1
    return torch.where(solid, -best.sqrt(), best.sqrt())


def _node_positions(n, grid4):
    g = torch.from_numpy(np.asarray(grid4)).double().cuda()
    axis = torch.arange(n, device="cuda", dtype=F64)
    p = torch.stack(torch.meshgrid(axis, axis, axis, indexing="ij"), -1).flip(-1).reshape(-1, 3)
    return p * g[3] + g[:3]


def _corners(n, cell):
    step = torch.tensor([(c & 1) + n * ((c >> 1 & 1) + n * (c >> 2)) for c in range(8)], device="cuda")
    return (cell[:, 0] + n * (cell[:, 1] + n * cell[:, 2]))[:, None] + step


def _interpolate(f, x):
    """Trilinear value of corner samples f (m, 8) at in-cell positions x (m, 3)."""
    f = f[:, 0::2] + x[:, :1] * (f[:, 1::2] - f[:, 0::2])
    f = f[:, 0::2] + x[:, 1:2] * (f[:, 1::2] - f[:, 0::2])
    return f[:, 0] + x[:, 2] * (f[:, 1] - f[:, 0])


def _first_root(values, n, grid4, o, d, lo, hi):
    """First t in [lo, hi] where the interpolant of the samples is <= 0, else
    inf, and the cell it lies in: cell by cell along every ray."""
    g = torch.from_numpy(np.asarray(grid4)).double().cuda()
    p, q = (o.double() - g[:3]) / g[3], d.double() / g[3]
    values = values.double()
    inv = 1 / torch.where(q == 0, 1e-300, q)
    near, far = torch.minimum(-p * inv, (n - 1 - p) * inv), torch.maximum(-p * inv, (n - 1 - p) * inv)
    lo, hi = torch.maximum(near.amax(1), lo), torch.minimum(far.amin(1), hi)
    found = torch.full_like(lo, math.inf)
    cells = torch.zeros(len(p), 3, dtype=torch.long, device="cuda")
    live = (lo <= hi).nonzero()[:, 0]
    cell = (p + lo[:, None] * q).floor().long().clamp(0, n - 2)[live]
    t = lo[live]
    while len(live):
        a, b = p[live], q[live]
        exits = torch.where(b == 0, math.inf, (cell + (b > 0) - a) * inv[live])
        t1, axis = exits.min(1)
        end = torch.minimum(torch.maximum(t1, t), hi[live])
        f = values[_corners(n, cell)]
        at = (f.amin(1) <= 0).nonzero()[:, 0]
        if len(at):
            fa, pa, qa, ta, tb = f[at], a[at] - cell[at], b[at], t[at], end[at]
            # the cubic along the ray from four values, its stationary points,
            # then bisection on the first piece that ends at or below zero
            s = torch.linspace(0, 1, 4, device="cuda", dtype=F64)
            y = [_interpolate(fa, pa + (ta + k * (tb - ta))[:, None] * qa) for k in s]
            c0 = y[0]
            c1 = -5.5 * y[0] + 9 * y[1] - 4.5 * y[2] + y[3]
            c2 = 9 * y[0] - 22.5 * y[1] + 18 * y[2] - 4.5 * y[3]
            c3 = -4.5 * y[0] + 13.5 * y[1] - 13.5 * y[2] + 4.5 * y[3]
            root = (c2 * c2 - 3 * c1 * c3).clamp(min=0).sqrt()
            w = -(c2 + torch.copysign(root, c2))
            k0, k1 = w / (3 * c3), c1 / w
            stops = torch.stack([k0, k1], 1).nan_to_num(1.0, 1.0, 1.0).clamp(0, 1).sort(1).values
            begin, stop = torch.zeros_like(c0), torch.full_like(c0, math.inf)
            for k in (begin, stops[:, 0], stops[:, 1], torch.ones_like(c0)):
                value = _interpolate(fa, pa + (ta + k * (tb - ta))[:, None] * qa)
                first = (value <= 0) & torch.isinf(stop)
                begin = torch.where((value > 0) & torch.isinf(stop), k, begin)
                stop = torch.where(first, k, stop)
            hit = torch.isfinite(stop)
            x0, x1 = begin, stop.clamp(max=1)
            for _ in range(54):
                mid = (x0 + x1) / 2
                below = _interpolate(fa, pa + (ta + mid * (tb - ta))[:, None] * qa) <= 0
                x0, x1 = torch.where(below, x0, mid), torch.where(below, mid, x1)
            rays = live[at[hit]]
            found[rays] = (ta + x1 * (tb - ta))[hit]
            cells[rays] = cell[at[hit]]
        move = torch.zeros_like(cell).scatter_(1, axis[:, None], torch.where(b > 0, 1, -1).gather(1, axis[:, None]))
        cell = cell + move
        stay = torch.isinf(found[live]) & (t1 < hi[live]) & (cell >= 0).all(1) & (cell <= n - 2).all(1)
        live, cell, t = live[stay], cell[stay], end[stay]
    return found, cells, p, q, lo


def _exact_trace(case, state):
    """The combined query (its field built from the mesh by brute force): t, then u and v."""
    o, d = state["rays"].T[:, :3], state["rays"].T[:, 3:]
    tri, zero = _mesh(*_key(case)), torch.zeros(len(o), device="cuda", dtype=F64)
    grid4 = workloads.room_grid(case["n"])
    split = min(float(np.float32(case["tau"] * float(grid4[3]))), case["tmax"])
    if case["kind"] == "bvh":
        split = case["tmax"]
    t, u, v = zero + math.inf, zero.clone(), zero.clone()
    if split > 0:
        for rays in torch.arange(len(o), device="cuda").split(max(1, (1 << 25) // len(tri))):
            k, a, b = _hit_triangles(o[rays, None].double(), d[rays, None].double(), tri[None])
            k, which = k.min(1)
            inside = k <= split
            t[rays] = torch.where(inside, k, math.inf)
            u[rays] = torch.where(inside, a.gather(1, which[:, None])[:, 0], 0.0)
            v[rays] = torch.where(inside, b.gather(1, which[:, None])[:, 0], 0.0)
    if case["kind"] == "trace":
        field = _mesh_distance(tri, _node_positions(case["n"], grid4), 1).float()
        field = field.half() if case["fmt"] == "f16" else field
        k = _first_root(field, case["n"], grid4, o, d, zero + split, zero + case["tmax"])[0]
        t = torch.where(torch.isinf(t), k, t)
    return t, None, u, v


def exact(case, seed):
    nodes, mesh = case["n"] ** 3, 0 if case["kind"] == "batch" else _scene(*_key(case)).n_tris
    rays = case["rays"] or case["width"] * case["height"] * case["spp"]
    if case["kind"] == "bvh":
        return _exact_trace(case, prepare(case, seed)) if mesh * rays <= 2e9 else None
    if case["kind"] == "trace":
        small = mesh <= 3000 and nodes * mesh <= 4e9 and mesh * rays <= 2e9
        return _exact_trace(case, prepare(case, seed)) if small and case["fmt"] != "i8" else None
    if case["kind"] in ("build", "load"):
        if mesh > 3000 or nodes * mesh > 4e9 or case["fmt"] == "i8":
            return None
        state = prepare(case, seed)
        tri = torch.from_numpy(state["verts"][state["tris"]]).cuda().double()
        out = _mesh_distance(tri, _node_positions(case["n"], state["grid4"]), 1).reshape((case["n"],) * 3)
        return out if case["fmt"] == "f32" else out.float().half().double()
    if case["kind"] not in ("refit", "update") or case["fmt"] == "i8":
        return None
    state, n = prepare(case, seed), case["n"]
    o, d = state["rays"].T[:, :3], state["rays"].T[:, 3:]
    values = state["values"].detach()
    values = (values.half() if case["fmt"] == "f16" else values).double()
    zero = torch.zeros(len(o), device="cuda", dtype=F64)
    t, cell, p, q, start = _first_root(values, n, state["grid4"], o, d, zero, zero + case["tmax"])
    if case["kind"] == "update":
        return t, None, zero, zero
    hit = (torch.isfinite(t) & (t > start)).nonzero()[:, 0]
    nodes = _corners(n, cell[hit])
    f, x = values[nodes], p[hit] + t[hit, None] * q[hit] - cell[hit]
    sign = torch.tensor([[1.0 if c >> k & 1 else -1.0 for k in range(3)] for c in range(8)], device="cuda", dtype=F64)
    weight = 0.5 + sign * (x[:, None] - 0.5)  # (m, 8, 3): the linear weight along each axis
    slope = 0
    for k in range(3):
        others = weight[..., (k + 1) % 3] * weight[..., (k + 2) % 3]
        slope = slope + (f * sign[:, k] * others).sum(1) * q[hit, k]
    share = -weight.prod(2) / slope[:, None] * state["grad_t"].double()[hit, None]
    grad = torch.zeros(n ** 3, device="cuda", dtype=F64)
    return t, grad.index_add_(0, nodes.reshape(-1), share.reshape(-1))
