"""GPU: what the choice of a traversal must not change: trees and launches on both sides of
the lines by size, closest and any hit, and shadow queries whose two triangle segments lie
on different sides of the line by length, against their three parts queried by themselves."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
CLOSEST, ANY = 2048, 8192  # triangles
LAUNCH = 1 << 19           # rays
G4 = np.array([-0.0625, -0.0625, -0.0625, 0.03125], np.float32)  # 37^3, a voxel a power of two


def mesh(count):
    """The first `count` triangles of a room with objects."""
    from paper_2305_07253_amd import workloads as W
    sc = W.make_scene(6, 120 if count < 5000 else 400, 0.01, 0.12, box_subdiv=2, ico_splits=1)
    assert len(sc.tris) >= count
    return sc.verts, sc.tris[:count]


def some_rays(n, seed=8):
    import torch
    rng = np.random.default_rng(seed)
    o, d = rng.random((n, 3)), rng.normal(size=(n, 3))
    d[:n // 60, rng.integers(3)] = 0.0
    d[n // 60:n // 50] = np.eye(3)[rng.integers(3, size=n // 50 - n // 60)]
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    return torch.from_numpy(np.ascontiguousarray(np.concatenate([o, d], 1).T.astype(np.float32))).cuda()


def same(a, b):
    import torch
    return all(torch.equal(x.view(torch.int32), y.view(torch.int32)) for x, y in zip(a, b))


@pytest.mark.parametrize("count", [CLOSEST, ANY])
def test_tree_size(count):
    """One triangle more, far away, does not change a hit."""
    import torch
    import paper_2305_07253_amd as hyb
    assert torch.cuda.is_available()
    verts, tris = mesh(count)
    far = np.concatenate([verts, np.float32([[50, 50, 50], [51, 50, 50], [50, 51, 50]])])
    more = np.concatenate([tris, np.int32([[0, 1, 2]]) + len(verts)])
    a, b = hyb.build_bvh(verts, tris), hyb.build_bvh(far, more)
    rays = some_rays(30011)
    assert same(hyb.trace_bvh(a, rays, 3.0), hyb.trace_bvh(b, rays, 3.0))
    for fmt in (0, 1, 2):
        sdf = hyb.build_sdf(a, 37, G4, fmt=fmt)
        for tau in (9.0, np.inf):
            assert same(hyb.trace(a, sdf, rays, 3.0, tau), hyb.trace(b, sdf, rays, 3.0, tau))
            got = [hyb.trace_shadow(x, sdf, rays, 1.0, tau, tau)[1] for x in (a, b)]
            # which occluder an any-hit query reports is open, that there is one is not
            assert torch.equal(got[0].clamp(max=0), got[1].clamp(max=0))


def test_launch_size():
    """The same rays in launches below and above the line, and few of them."""
    import torch
    import paper_2305_07253_amd as hyb
    assert torch.cuda.is_available()
    bvh = hyb.build_bvh(*mesh(CLOSEST))
    sdf = hyb.build_sdf(bvh, 37, G4)
    rays = some_rays(LAUNCH + 1)
    for query in (lambda r: hyb.trace_bvh(bvh, r, 3.0), lambda r: hyb.trace(bvh, sdf, r, 3.0, 9.0)):
        whole = query(rays)
        for n in (77, 40001, LAUNCH):
            assert same(query(rays[:, :n].contiguous()), [x[:n] for x in whole])


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("count", [CLOSEST, ANY, ANY + 1])
@pytest.mark.parametrize("start, end", [(4.0, 4.0), (4.0000005, 4.0000005), (4.0, 4.0000005), (4.0000005, 4.0),
                                        (0.0, 9.0), (9.0, 0.0), (2.5, 30.0)])
def test_shadow_is_its_three_parts(fmt, count, start, end):
    import torch
    import paper_2305_07253_amd as hyb
    assert torch.cuda.is_available()
    bvh = hyb.build_bvh(*mesh(count))
    sdf = hyb.build_sdf(bvh, 37, G4, fmt=fmt)
    rays = some_rays(20011)
    tmax, h = np.float32(1.0), np.float64(G4[3])
    t1 = min(np.float32(np.float32(start) * h), tmax)
    t2 = max(np.float32(tmax - np.float64(np.float32(end)) * h), t1)
    n = rays.shape[1]
    at1, at2 = (torch.full((n,), float(t), device="cuda") for t in (t1, t2))
    miss = torch.zeros(n, dtype=torch.bool, device="cuda")
    near = hyb.trace_bvh(bvh, rays, float(t1))[1] >= 0 if t1 > 0 else miss
    far = hyb.trace_bvh(bvh, rays, float(tmax), tmin=at2)[1] >= 0 if t2 < tmax else miss
    field_t, field = hyb.trace_df(sdf, rays, float(t2), tmin=at1)[:2]
    field = field == -2 if t2 > t1 else miss
    t, prim = hyb.trace_shadow(bvh, sdf, rays, float(tmax), start, end)[:2]
    assert torch.equal(prim == -2, field)
    assert torch.equal(t[field], field_t[field])
    assert torch.equal(prim >= 0, (near | far) & ~field)
    assert (near | far).any() and not (near & far).all()
