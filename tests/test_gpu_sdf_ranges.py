"""GPU: the distance-field build over the sizes and scales it takes, against the per-node
body on the CPU, which searches the tree in FP64 for each node by itself."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def check(verts, tris, n, g4, exterior=True):
    import torch
    import paper_2305_07253_amd as hyb
    from tests.emu import runner
    assert torch.cuda.is_available()
    got = hyb.sdf_read(hyb.build_sdf(hyb.build_bvh(verts, tris), n, g4, exterior_solid=exterior)).cpu().numpy()
    ref = runner.sdf(verts, tris, g4, n, exterior_solid=exterior)
    # the same FP64 steps but for contraction and a reciprocal: the FP32 rounding may differ
    assert np.all(np.abs(got.astype(np.float64) - ref) <= np.spacing(np.abs(ref)))


def loose(count, size, seed):
    rng = np.random.default_rng(seed)
    v = rng.random((count, 1, 3)) + size * (rng.random((count, 3, 3)) - 0.5)
    return v.astype(np.float32).reshape(-1, 3), np.arange(3 * count, dtype=np.int32).reshape(-1, 3)


@pytest.mark.parametrize("scale", [1.0, 1e-18, 1e-20, 1e-21, 3e-22])
@pytest.mark.parametrize("count", [3, 40])
@pytest.mark.parametrize("n", [12, 48])
def test_squares_below_the_normal_range(scale, count, n):
    """Distances whose squares FP32 holds to a few bits only, or not at all."""
    verts, tris = loose(count, 0.4, 5)
    g4 = np.array([-0.1, -0.1, -0.1, 1.2 / (n - 1)], np.float32) * np.float32(scale)
    check(verts * np.float32(scale), tris, n, g4)


@pytest.mark.parametrize("n, line", [(8, 1.0), (9, 1.0), (27, 1.0), (40, 1.0), (41, 6.15), (50, 7.5)])
@pytest.mark.parametrize("side", [0.98, 1.02])
@pytest.mark.parametrize("mesh", ["closed", "loose"])
def test_both_searches(n, line, side, mesh):
    """Grids on both sides of the line between packets of nodes and nodes by themselves (a
    voxel in triangles of a surface that spans the mesh), with wavefronts not filled."""
    from paper_2305_07253_amd import workloads as W
    scene = W.make_scene(4, 6, 0.05, 0.2, box_subdiv=1, ico_splits=1)
    verts, tris = (scene.verts, scene.tris) if mesh == "closed" else loose(150, 0.3, 9)
    lo, extent = verts.min(0), float((verts.max(0) - verts.min(0)).max())
    h = side * line * extent / len(tris) ** 0.5
    g4 = np.append(lo + (0.37 * extent - 0.5 * h * (n - 1)), h).astype(np.float32)
    check(verts, tris, n, g4, exterior=n % 2 == 0)


def test_detailed_mesh_on_coarse_grid():
    """Long searches: deep stacks, many boxes and triangles for each node."""
    from paper_2305_07253_amd import workloads as W
    scene = W.make_scene(5, 60, 0.01, 0.12, box_subdiv=4, ico_splits=2)
    check(scene.verts, scene.tris, 17, W.room_grid(17))


@pytest.mark.parametrize("n", [8, 13, 33])
@pytest.mark.parametrize("count", [0, 1, 2, 31, 32, 33])
def test_few_triangles(count, n):
    """Around the count up to which one pass goes through all triangles for every node."""
    verts, tris = loose(count, 0.4, count)
    g4 = np.array([-0.2, -0.1, -0.15, 1.3 / (n - 1)], np.float32)
    if count == 0:
        import paper_2305_07253_amd as hyb
        with pytest.raises(hyb.HybError):  # every sample is infinite
            hyb.build_sdf(hyb.build_bvh(verts, tris), n, g4)
        return
    for exterior in (True, False):
        check(verts, tris, n, g4, exterior)


def test_walls_alone():
    """A closed mesh of few triangles: solid outside, or inside once it is turned."""
    from paper_2305_07253_amd import workloads as W
    scene = W.make_scene(1, 1, 0.2, 0.3, box_subdiv=1, ico_splits=1)
    walls = scene.tris[:12]
    for tris in (walls, np.ascontiguousarray(walls[:, ::-1])):
        for exterior in (True, False):
            check(scene.verts, tris, 19, W.room_grid(19), exterior)
