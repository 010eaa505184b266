"""GPU: the traversals for short and long triangle segments, and the batch's own,
give a ray one result: thresholds on both sides of the rule's line, against the
triangles-only query and the same rays in a batch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("below, above", [(4.0, 4.0000005), (0.0, 1e30)])
def test_hits_do_not_depend_on_the_traversal(fmt, below, above):
    import torch
    import paper_2305_07253_amd as hyb
    from paper_2305_07253_amd import workloads as W
    assert torch.cuda.is_available()
    sc = W.make_scene(6, 60, 0.01, 0.12)
    bvh = hyb.build_bvh(sc.verts, sc.tris)
    sdf = hyb.build_sdf(bvh, 40, W.room_grid(40), fmt=fmt)
    h = float(W.room_grid(40)[3])
    rng = np.random.default_rng(8)
    n = 30011
    o, d = rng.random((n, 3)), rng.normal(size=(n, 3))
    d[:500, rng.integers(3)] = 0.0
    d[500:600] = np.eye(3)[rng.integers(3, size=100)] * rng.choice([-1.0, 1.0], (100, 1))
    d = d.astype(np.float32)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rays = torch.from_numpy(np.ascontiguousarray(np.concatenate([o, d], 1).T.astype(np.float32))).cuda()
    for tau in (below, above):
        got = hyb.trace(bvh, sdf, rays, 1.0, tau)
        batch = hyb.Batch([dict(bvh=bvh, sdf=sdf, rays=rays, tmax=1.0, threshold=tau)]).launch()[0]
        for a, b in zip(got, batch):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))
        # a triangle hit of the combined query is the one that triangles alone give
        ref = hyb.trace_bvh(bvh, rays, min(float(np.float32(np.float32(tau) * np.float32(h))), 1.0))
        near = ref[1] >= 0
        assert torch.equal(got[1] >= 0, near)
        for a, b in zip(got, ref):
            assert torch.equal(a[near], b[near])
        # any hit: occluded exactly where some segment is
        t, prim, _, _ = hyb.trace_shadow(bvh, sdf, rays, 1.0, tau, tau)
        if tau >= 1.0 / h:
            assert torch.equal(prim >= 0, near)
    counts = [hyb.trace_counters(bvh, sdf, rays, 1.0, tau)[1][:, 1] for tau in (4.0, 4.0000005)]
    assert (counts[0] > 0).any() and (counts[1] > 0).any()
