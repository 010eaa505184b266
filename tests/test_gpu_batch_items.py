"""GPU: how a batch cuts its rays into work items: fewer rays than a wavefront holds in
small batches, one wavefront's, and more than 2^20 wavefronts of them; item counts around
the 64-way search for a work item's scene; empty items first, last and in between."""
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
    return hyb, bvh, sdf, rays, [x.cpu().numpy() for x in hyb.trace(bvh, sdf, rays, 2.0, 1.0)]


@pytest.mark.parametrize("n_items, rays", [(1, 1), (1, 63), (3, 2048), (3, 2049), (64, 4096), (65, 4097), (64, 65537),
                                           (129, 131072), (4097, 131073), (4160, 1 << 18), (65, 1 << 18)])
@pytest.mark.parametrize("static", [False, True], ids=["handle", "static"])
def test_items_cover_every_ray_once(room, n_items, rays, static):
    hyb, bvh, sdf, all_rays, want = room
    if static and n_items > 256:
        n_items = 256
    rng = np.random.default_rng(n_items + rays)
    # uneven runs, a third of them empty where there are several
    cuts = np.sort(rng.integers(0, rays + 1, n_items - 1))
    cuts[rng.random(n_items - 1) < 0.33] = 0
    cuts = np.concatenate([[0], np.sort(cuts), [rays]])
    items = [dict(bvh=bvh, sdf=sdf, rays=all_rays[:, a:b].contiguous(), tmax=2.0, threshold=1.0)
             for a, b in zip(cuts[:-1], cuts[1:])]
    config = dict(lds_depth=16, rays_per_item=192, blocks_per_cu=4)
    if static:
        runs = [hyb.batch_launch_static(items), hyb.batch_launch_static(items, config)]
    else:
        batch = hyb.Batch(items)
        runs = [batch.launch(), batch.launch(graph=False)]
        batch.config = config
        runs.append(batch.launch())
    for outs in runs:
        for k in range(4):
            got = np.concatenate([o[k].cpu().numpy() for o in outs])
            assert np.array_equal(got, want[k][:rays])


@pytest.mark.parametrize("rays_per_item", [64, 192, 256])
def test_more_than_a_million_wavefronts(room, rays_per_item):
    """2^26 + 2^18 rays: 257 items that share their rays and hit buffers."""
    import torch
    hyb, bvh, sdf, rays, want = room
    n = rays.shape[1]
    out = (torch.empty(n, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda"),
           torch.empty(n, device="cuda"), torch.empty(n, device="cuda"))
    batch = hyb.Batch([dict(bvh=bvh, sdf=sdf, rays=rays, tmax=2.0, threshold=1.0, out=out)] * 257)
    batch.config = dict(lds_depth=16, rays_per_item=rays_per_item, blocks_per_cu=4)
    batch.launch()
    for k in range(4):
        assert np.array_equal(out[k].cpu().numpy(), want[k])
