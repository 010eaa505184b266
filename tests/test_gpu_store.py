"""GPU: the stored forms of a grid at the edges of the store kernel's tiles (32 x 8
x 4 cells) and of the I8 scale blocks: the samples as the kernels see them and
the Lipschitz bound, of new grids and of updates; the bricks through the field
that a dense set of short rays meets."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", [0, 1, 2])
@pytest.mark.parametrize("n", [2, 3, 5, 6, 8, 9, 10, 17, 32, 33, 34, 41, 65, 66, 206])
def test_samples_bounds_and_bricks(orc, n, fmt):
    import torch
    import paper_2305_07253_amd as hyb
    assert torch.cuda.is_available()
    rng = np.random.default_rng(n)
    g4 = np.array([0.25, -1.0, 2.0, 0.5], np.float32)
    before = rng.normal(size=(n, n, n)).astype(np.float32)
    values = (rng.normal(size=(n, n, n)) * rng.choice([1e-3, 1.0, 50.0], (n, n, n))).astype(np.float32)
    want = orc.quantize(values, fmt)[0]
    x = torch.from_numpy(values.reshape(-1)).cuda()
    sdf = hyb.sdf_from_grid(x, g4, fmt=fmt)
    waited = hyb.sdf_update(hyb.sdf_from_grid(torch.from_numpy(before.reshape(-1)).cuda(), g4, fmt=fmt), x)
    queued = hyb.sdf_update(hyb.sdf_from_grid(torch.from_numpy(before.reshape(-1)).cuda(), g4, fmt=fmt), x,
                            deferred=True)
    f = want.astype(np.float64)
    d = [np.abs(np.diff(f, axis=a)) for a in (2, 1, 0)]
    m = n - 1
    pairs = [(a, b) for a in (0, 1) for b in (0, 1)]  # the four edges of a cell along each axis
    ex = np.maximum.reduce([d[0][a:a + m, b:b + m] for a, b in pairs])
    ey = np.maximum.reduce([d[1][a:a + m, :, b:b + m] for a, b in pairs])
    ez = np.maximum.reduce([d[2][:, a:a + m, b:b + m] for a, b in pairs])
    bound = max(np.sqrt(ex ** 2 + ey ** 2 + ez ** 2).max() / 0.5, 1.0)
    # a ray down the middle of every cell column whose ends straddle it, per axis x
    cells = np.stack(np.meshgrid(np.arange(m), np.arange(m), np.arange(m), indexing="ij"), -1).reshape(-1, 3)
    cells = cells[rng.permutation(len(cells))[:20000]]
    o = (g4[:3] + 0.5 * (cells + [0.0, 0.37, 0.61])).astype(np.float32)
    rays = torch.from_numpy(np.ascontiguousarray(np.concatenate([o, np.tile(np.float32([1, 0, 0]), (len(o), 1))], 1).T)
                            ).cuda()
    # along x the interpolant is linear in a cell: from g0 at its start to g1 at its end
    c = {(a, b, e): f[cells[:, 2] + e, cells[:, 1] + b, cells[:, 0] + a] for a in (0, 1) for b in (0, 1) for e in (0, 1)}
    g = [(1 - 0.61) * ((1 - 0.37) * c[a, 0, 0] + 0.37 * c[a, 1, 0]) + 0.61 * ((1 - 0.37) * c[a, 0, 1] + 0.37 * c[a, 1, 1])
         for a in (0, 1)]
    scale = np.maximum.reduce([np.abs(v) for v in c.values()])
    clear = (np.abs(g[0]) > 1e-4 * scale) & (np.abs(g[1]) > 1e-4 * scale)
    hit = (g[0] <= 0) | (g[1] <= 0)
    for s in (sdf, waited, queued):
        assert np.array_equal(hyb.sdf_read(s).cpu().numpy(), want)
        # rounded up by 4e-7 and a few FP32 roundings
        assert bound <= s.lipschitz <= bound * (1 + 2e-6)
        prim = hyb.trace_df(s, rays, 0.5 * (1 - 1e-6))[1].cpu().numpy()
        assert np.array_equal((prim == -2)[clear], hit[clear])
