"""GPU: launches of few rays spread them over more wavefronts, several lanes to
a ray.  Each ray's result is the one it has in a launch that fills the chip."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 1024, 1025, 2047, 2049, 4097, 8192, 8193, 16385, 65536, 65537, 131071, 131073])
def test_results_do_not_depend_on_the_launch_size(n):
    import torch
    import paper_2305_07253_amd as hyb
    from paper_2305_07253_amd import workloads as W
    assert torch.cuda.is_available()
    sc = W.tiny_scene(1)
    bvh = hyb.build_bvh(sc.verts, sc.tris)
    rng = np.random.default_rng(4)
    o = rng.random((200000, 3))
    d = rng.normal(size=(200000, 3)).astype(np.float32)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rays = np.concatenate([o, d], 1).T.astype(np.float32)
    every = torch.from_numpy(np.ascontiguousarray(rays)).cuda()
    some = torch.from_numpy(np.ascontiguousarray(rays[:, -n:])).cuda()
    lengths = torch.linspace(0.0, 1.5, every.shape[1], device="cuda")
    for fmt in (hyb.SDF_F32, hyb.SDF_F16, hyb.SDF_I8_BRICK):
        sdf = hyb.build_sdf(bvh, 32, W.room_grid(32), fmt=fmt)
        for query in (lambda r, t: hyb.trace(bvh, sdf, r, 2.0, 1.0, tmax_ray=t),
                      lambda r, t: hyb.trace(bvh, sdf, r, 2.0, 0.0, tmax_ray=t),
                      lambda r, t: hyb.trace_bvh(bvh, r, 2.0, tmax_ray=t),
                      lambda r, t: hyb.trace_shadow(bvh, sdf, r, 2.0, 1.0, 1.0, tmax_ray=t)):
            for got, ref in zip(query(some, lengths[-n:].contiguous()), query(every, lengths)):
                assert torch.equal(got.view(torch.int32), ref[-n:].view(torch.int32))
        got, counts = hyb.trace_counters(bvh, sdf, some, 2.0, 1.0)
        ref, ref_counts = hyb.trace_counters(bvh, sdf, every, 2.0, 1.0)
        assert torch.equal(counts, ref_counts[-n:]) and torch.equal(got[1], ref[1][-n:])
