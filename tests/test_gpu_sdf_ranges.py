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
