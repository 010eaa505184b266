"""GPU: sums of the backward at the sizes where its kernels change: workgroups of 512
rays, the line at 2^18 rays above which the rays are sorted, blocks of 8^3 cells that
end on, before and after the grid does, and workgroups that hold more than 32 blocks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
LINE = 1 << 18


@pytest.mark.parametrize("n, rays", [(n, m) for n in (2, 9, 10, 17, 18, 64) for m in (1, 512, 513, LINE, LINE + 1)]
                         + [(264, LINE), (264, LINE + 1)])
def test_sums_of_exact_crossings(n, rays):
    """Layers of period 8 along z, exact in FP32 and linear within every cell: rays
    that start up to half a cell before a layer's middle, so that t and its
    derivatives are known, each with a grad_t of its own."""
    import torch
    import paper_2305_07253_amd as hyb
    assert torch.cuda.is_available()
    rng = np.random.default_rng(n * 7 + rays)
    h = 0.0625
    g4 = np.array([0.0, 0.0, 0.0, h], np.float32)
    layer = h * (np.abs((np.arange(n) + 1) % 8 - 4.0) - 2.5)
    field = torch.from_numpy(layer.astype(np.float32)).cuda().repeat_interleave(n * n)
    sdf = hyb.sdf_from_grid(field, g4)

    # crossings upward at z = 8 k + 0.5 cells, downward at 8 k - 2.5
    up = np.arange(0, n - 1, 8)
    down = np.arange(8, n + 2, 8)
    down = down[down - 2 <= n - 1]
    pick = rng.integers(0, len(up) + len(down), rays)
    rise = pick < len(up)
    at = np.where(rise, np.concatenate([up, down])[pick] + 0.5, np.concatenate([up, down])[pick] - 2.5)
    x, y = (rng.integers(0, n - 1, rays) + rng.uniform(0.15, 0.85, rays) for _ in range(2))
    back = rng.uniform(0.1, 0.45, rays)
    o = np.stack([x, y, at + np.where(rise, -back, back)], 1) * h
    d = np.stack([*rng.uniform(-0.2, 0.2, (2, rays)), np.where(rise, 1.0, -1.0)], 1)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    r32 = np.ascontiguousarray(np.concatenate([o, d], 1).T.astype(np.float32))
    gt = rng.normal(size=rays).astype(np.float32)

    r = r32.astype(np.float64)
    t = (at * h - r[2]) / r[5]
    p = (r[:3] + t * r[3:]) / h
    cell = np.floor(p).astype(np.int64)
    assert (cell >= 0).all() and (cell < n - 1).all()
    f = p - cell
    want, weight, count = (np.zeros(n ** 3) for _ in range(3))
    for c in range(8):
        bit = [(c >> a) & 1 for a in range(3)]
        w = np.prod([f[a] if bit[a] else 1 - f[a] for a in range(3)], axis=0)
        node = cell[0] + bit[0] + n * (cell[1] + bit[1] + n * (cell[2] + bit[2]))
        # the layer falls by h a cell along the ray: grad . d = -|dz|
        np.add.at(want, node, gt * w / np.abs(r[5]))
        np.add.at(weight, node, np.abs(gt))
        np.add.at(count, node, 1)
    # a point's FP32 rounding, 4 units of a coordinate up to n cells, moves each of three
    # weights; 1e-5 for the derivative's own roundings; the order of the additions
    tol = weight * (12 * n * 2.0 ** -23 + 1e-5 + count * 2.0 ** -24) + 1e-30

    dev = torch.from_numpy(r32).cuda()
    hit, prim = hyb.trace_df(sdf, dev, 2 * h)[:2]
    assert (prim == -2).all()
    for start in (0.0, 0.5):  # added to what is there
        grad = torch.full((n ** 3,), start, device="cuda")
        hyb.df_backward(sdf, dev, 2 * h, hit, torch.from_numpy(gt).cuda(), grad)
        got = grad.cpu().numpy().astype(np.float64) - start
        assert (np.abs(got - want) <= tol + start * (count + 1) * 2.0 ** -23).all()
        assert (got[count == 0] == 0).all()
