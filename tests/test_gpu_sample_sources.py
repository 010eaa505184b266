"""GPU: where the samples of a grid may lie: device memory, also inside an allocation, and
host memory, pinned or not; a buffer of fewer samples than the grid has is an error."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def status(hyb, address, n, g4, fmt, sdf=None):
    """(status, handle) of hyb_sdf_from_grid, or of hyb_sdf_update where sdf is given."""
    import torch
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    if sdf is not None:
        return hyb.lib().hyb_sdf_update(sdf.handle, ctypes.c_void_p(address), 0, stream), None
    out = ctypes.c_void_p()
    rc = hyb.lib().hyb_sdf_from_grid(ctypes.c_void_p(address), n, g4.ctypes.data_as(ctypes.c_void_p), 0, fmt, stream,
                                     ctypes.byref(out))
    return rc, out


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("n", [5, 40])
def test_sources(fmt, n):
    import torch
    import paper_2305_07253_amd as hyb
    assert torch.cuda.is_available()
    rng = np.random.default_rng(n)
    g4 = np.array([0, 0, 0, 1.0 / n], np.float32)
    host = rng.random((2, n, n, n), dtype=np.float32) - np.float32(0.4)
    dev = torch.from_numpy(host).cuda()
    pinned = torch.empty(host.shape, dtype=torch.float32, pin_memory=True)
    pinned.copy_(torch.from_numpy(host))
    inside = torch.empty(3 + host.size, device="cuda")
    inside[3:] = dev.reshape(-1)
    sources = [dev.data_ptr(), inside.data_ptr() + 12, pinned.data_ptr(), host.ctypes.data]
    want = [hyb.sdf_read(hyb.sdf_from_grid(dev[k].reshape(-1), g4, fmt=fmt)) for k in (0, 1)]
    bounds = [hyb.sdf_from_grid(dev[k].reshape(-1), g4, fmt=fmt).lipschitz for k in (0, 1)]
    for at in sources:
        rc, handle = status(hyb, at, n, g4, fmt)
        assert rc == 0
        sdf = hyb.Sdf(handle)
        assert torch.equal(hyb.sdf_read(sdf), want[0]) and sdf.lipschitz == bounds[0]
        rc, _ = status(hyb, at + 4 * n ** 3, n, g4, fmt, sdf)
        assert rc == 0
        assert torch.equal(hyb.sdf_read(sdf), want[1]) and sdf.lipschitz == bounds[1]


def test_too_few_samples():
    """64 MiB where 2 GiB are needed (an allocation of its own, larger than any it could be
    part of)."""
    import torch
    import paper_2305_07253_amd as hyb
    assert torch.cuda.is_available()
    torch.cuda.empty_cache()
    few = torch.zeros(1 << 24, device="cuda")
    rc, _ = status(hyb, few.data_ptr(), 813, np.array([0, 0, 0, 1], np.float32), 0)
    assert rc != 0
