"""GPU: the distance-field build at the edges of its tiles (4^3 nodes a
wavefront, 8^3 nodes a component block), on closed and open meshes, against the
same build's definition: exact distances, sign by winding number."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def winding_distance(verts, tris, grid4, n, exterior):
    """Signed distance of every node by brute force in FP64 ([k, j, i]): nearest
    triangle, and signed crossings of one ray per node."""
    axis = float(grid4[3]) * np.arange(n)
    p = np.stack(np.meshgrid(float(grid4[2]) + axis, float(grid4[1]) + axis, float(grid4[0]) + axis, indexing="ij"),
                 -1)[..., ::-1].reshape(-1, 3)
    best, wind = np.full(len(p), np.inf), np.full(len(p), int(exterior))
    D = np.array([0.61, 0.5177, 0.6003])
    D /= np.linalg.norm(D)
    for a, b, c in verts.astype(np.float64)[tris]:
        m = np.cross(b - a, c - a)
        inside = np.ones(len(p), bool)
        for s, e in ((a, b), (b, c), (c, a)):
            w, edge = p - s, e - s
            k = np.clip(w @ edge / (edge @ edge), 0, 1) if edge @ edge > 0 else np.zeros(len(p))
            best = np.minimum(best, ((w - k[:, None] * edge) ** 2).sum(1))
            inside &= w @ np.cross(m, edge) >= 0
        if m @ m > 0:
            best = np.where(inside, np.minimum(best, ((p - a) @ m) ** 2 / (m @ m)), best)
            x, y, z = a - p, b - p, c - p
            u, v, w = np.cross(y, z) @ D, np.cross(z, x) @ D, np.cross(x, y) @ D
            hit = ((u >= 0) & (v >= 0) & (w >= 0)) | ((u <= 0) & (v <= 0) & (w <= 0))
            if D @ m != 0:
                wind += np.where(hit & (u + v + w != 0) & (x @ m / (D @ m) > 0), int(np.sign(D @ m)), 0)
    return np.where(wind >= 1, -np.sqrt(best), np.sqrt(best)).reshape(n, n, n)


def meshes():
    from paper_2305_07253_amd import workloads as W
    box = W.make_scene(3, 6, 0.05, 0.2, box_subdiv=1, ico_splits=1)
    rng = np.random.default_rng(2)
    soup = rng.random((9, 3, 3)).astype(np.float32)
    return {"closed": (box.verts, box.tris), "a triangle left out": (box.verts, np.delete(box.tris, 20, 0)),
            "vertices not shared": (box.verts[box.tris].reshape(-1, 3),
                                    np.arange(3 * len(box.tris), dtype=np.int32).reshape(-1, 3)),
            "inside out": (box.verts, np.ascontiguousarray(box.tris[:, ::-1])),
            "loose triangles": (soup.reshape(-1, 3), np.arange(27, dtype=np.int32).reshape(9, 3)),
            "zero-area triangles": (box.verts, np.concatenate([box.tris, [[1, 1, 3], [2, 2, 2]]]).astype(np.int32))}


@pytest.mark.parametrize("exterior", [True, False])
@pytest.mark.parametrize("n", [8, 9, 12, 23])
@pytest.mark.parametrize("name", ["closed", "a triangle left out", "vertices not shared", "inside out",
                                  "loose triangles", "zero-area triangles"])
def test_build_is_the_winding_distance(name, n, exterior):
    import torch
    import paper_2305_07253_amd as hyb
    assert torch.cuda.is_available()
    verts, tris = meshes()[name]
    g4 = np.array([-0.13, -0.21, -0.17, 1.37 / (n - 1)], np.float32)
    got = hyb.sdf_read(hyb.build_sdf(hyb.build_bvh(verts, tris), n, g4, exterior_solid=exterior)).cpu().numpy()
    ref = winding_distance(verts, tris, g4, n, exterior)
    # one rounding of the FP64 distance, itself good to a few units of 2^-52
    assert np.all(np.abs(got.astype(np.float64) - ref) <= np.spacing(np.abs(ref).astype(np.float32)))
