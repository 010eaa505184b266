"""GPU: the traversal entry pyramid built on the device.  A segment of at most
eight finest voxels starts at its window's entry, a longer one at the root, so
a wrong entry would lose hits of the short segment that the long one finds.
(Segments begin a little after the ray's origin: a triangle within FP32
rounding of the begin may pass the triangle test yet fail the test of the box
around it, which only a traversal that begins above the leaf does.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def meshes():
    from paper_2305_07253_amd import workloads as W
    rng = np.random.default_rng(5)
    tiny = W.tiny_scene(1)
    soup = rng.random((60, 3, 3)).astype(np.float32)  # boxes as large as the whole mesh
    flat = rng.random((40, 3, 3)).astype(np.float32)
    flat[..., 2] = 0.25
    scene = W.make_scene(9, 40, 0.01, 0.1)
    return {"tiny": (tiny.verts, tiny.tris),
            "one triangle": (np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0]], np.float32), np.array([[0, 1, 2]], np.int32)),
            "five triangles": (soup[:5].reshape(-1, 3), np.arange(15, dtype=np.int32).reshape(5, 3)),
            "large triangles": (soup.reshape(-1, 3), np.arange(180, dtype=np.int32).reshape(60, 3)),
            "flat": (flat.reshape(-1, 3), np.arange(120, dtype=np.int32).reshape(40, 3)),
            "far off": (scene.verts * np.float32(30) + np.float32(500), scene.tris)}


@pytest.mark.parametrize("name", ["tiny", "one triangle", "five triangles", "large triangles", "flat", "far off"])
def test_short_segments_find_what_long_ones_do(name):
    import torch
    import paper_2305_07253_amd as hyb
    verts, tris = meshes()[name]
    bvh = hyb.build_bvh(verts, tris)
    lo, ext = verts.min(0), float((verts.max(0) - verts.min(0)).max())
    voxel = ext / 64
    rng = np.random.default_rng(7)
    n = 200000
    # starts on, near and around the mesh
    on = verts[tris[rng.integers(len(tris), size=n)]]
    w = rng.dirichlet((1, 1, 1), n)
    o = (on * w[..., None]).sum(1) + rng.normal(size=(n, 3)) * voxel * rng.choice([1e-3, 0.3, 2.0], (n, 1))
    o[: n // 8] = lo + ext * (rng.random((n // 8, 3)) * 1.2 - 0.1)
    d = rng.normal(size=(n, 3)).astype(np.float32)
    d[: n // 50, 1] = 0.0
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rays = torch.from_numpy(np.ascontiguousarray(np.concatenate([o, d], 1).T.astype(np.float32))).cuda()
    begin = torch.full((n,), 1e-2 * voxel, device="cuda")
    full = hyb.trace_bvh(bvh, rays, 12 * voxel, tmin=begin)
    for voxels in (0.05, 0.4, 0.9, 2.5, 7.9):
        got = hyb.trace_bvh(bvh, rays, voxels * voxel, tmin=begin)
        near = full[0] <= np.float32(voxels * voxel)
        assert near.any()
        assert torch.equal(got[1], torch.where(near, full[1], -1)), (name, voxels)
        for k in (0, 2, 3):
            assert torch.equal(got[k][near], full[k][near])
        assert torch.isinf(got[0][~near]).all()
