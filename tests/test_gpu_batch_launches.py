"""GPU: work items of large batches each checked by their own outputs, a second launch on
cleared outputs, and the launch tuner's choice of work items."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def room():
    import torch
    import paper_2305_07253_amd as hyb
    from paper_2305_07253_amd import workloads as W
    assert torch.cuda.is_available()
    scene = W.make_scene(3, 30, 0.03, 0.1, box_subdiv=1, ico_splits=1)
    bvh = hyb.build_bvh(scene.verts, scene.tris)
    sdf = hyb.build_sdf(bvh, 24, W.room_grid(24))
    rays = torch.from_numpy(np.ascontiguousarray(W.uniform_rays(scene, 1 << 18, 4).soa())).cuda()
    return hyb, bvh, sdf, rays, hyb.trace(bvh, sdf, rays, 2.0, 1.0)


def buffers(n):
    import torch
    return (torch.full((n,), -7.0, device="cuda"), torch.full((n,), -7, dtype=torch.int32, device="cuda"),
            torch.full((n,), -7.0, device="cuda"), torch.full((n,), -7.0, device="cuda"))


@pytest.mark.parametrize("rays_per_item", [64, 192, 256])
def test_every_item_of_a_large_batch(room, rays_per_item):
    """2^26 + 2^18 rays in 257 items with outputs of their own: around the 2^20th work item,
    at both ends and in between, in two launches."""
    import torch
    hyb, bvh, sdf, rays, want = room
    n = rays.shape[1]
    outs = [buffers(n) for _ in range(257)]
    batch = hyb.Batch([dict(bvh=bvh, sdf=sdf, rays=rays, tmax=2.0, threshold=1.0, out=out) for out in outs])
    batch.config = dict(lds_depth=16, rays_per_item=rays_per_item, blocks_per_cu=4)
    for graph in (True, False):
        batch.launch(graph=graph)
        for out in outs:
            assert all(torch.equal(a, b) for a, b in zip(out, want))
            for x in out:
                x.fill_(-7)


@pytest.mark.parametrize("items", [1, 5])
def test_tuner_times_each_launch_once(room, items):
    """Rays per item change nothing for a batch of this size: the smallest is reported."""
    import torch
    hyb, bvh, sdf, rays, want = room
    part = rays[:, :5000].contiguous()
    batch = hyb.Batch([dict(bvh=bvh, sdf=sdf, rays=part, tmax=2.0, threshold=1.0)] * items)
    for _ in range(3):
        batch.tune(0.0, threshold=False, reps=1)
        assert batch.config["rays_per_item"] == 64
    for out in batch.launch():
        assert all(torch.equal(a, b[:5000]) for a, b in zip(out, want))
