"""Distances to slivers (a vertex within an ulp of the opposite edge, down to one FP32
ulp of height) against exact rational arithmetic: grid rows that run along the triangle's
long edge and past its ends, and lattices that begin beyond an end of a slanted one.  The
per-node body on the CPU, and the build on the GPU."""
from fractions import Fraction

import numpy as np
import pytest

N = 8
F = np.float32


def squared_distance(p, a, b, c):
    """Squared distance of a point to a triangle, all coordinates Fractions."""
    def sub(x, y):
        return [i - j for i, j in zip(x, y)]

    def dot(x, y):
        return sum(i * j for i, j in zip(x, y))

    def cross(x, y):
        return [x[1] * y[2] - x[2] * y[1], x[2] * y[0] - x[0] * y[2], x[0] * y[1] - x[1] * y[0]]

    n = cross(sub(b, a), sub(c, a))
    ends = ((a, b), (b, c), (c, a))
    if any(n) and all(dot(cross(n, sub(t, s)), sub(p, s)) >= 0 for s, t in ends):
        return dot(sub(p, a), n) ** 2 / dot(n, n)
    best = None
    for s, t in ends:
        w, e = sub(p, s), sub(t, s)
        k = min(max(dot(w, e) / dot(e, e), Fraction(0)), Fraction(1)) if any(e) else Fraction(0)
        d = sum((i - k * j) ** 2 for i, j in zip(w, e))
        best = d if best is None else min(best, d)
    return best


def slivers():
    """(triangle, grid4) pairs; a grid's nodes are its own doubles, lo + i h exactly."""
    rng = np.random.default_rng(20)
    out = []
    for k in range(24):
        # an edge along an axis, the third vertex one ulp off it, and nodes on its line
        axis, side = k % 3, (k + 1 + k // 3 % 2) % 3
        a, b = rng.uniform(-0.5, 0.5, (2, 3)).astype(F)
        b = np.where(np.arange(3) == axis, b, a)
        c = a.copy()
        c[axis] = F(a[axis] + (b[axis] - a[axis]) * F(rng.uniform(0.1, 0.9)))
        c[side] = np.nextafter(a[side], F(2 if k % 2 else -2))
        lo = a.copy()
        lo[axis] = F(max(a[axis], b[axis]) + F(rng.uniform(0.01, 0.2)) if k % 4 else min(a[axis], b[axis]) - F(0.3))
        out.append((np.roll(np.stack([a, b, c]), k // 6, 0), np.append(lo, F(2.0 ** -rng.integers(3, 8)))))
    for k in range(24):
        # a slanted edge, the third vertex the nearest to a point of it, and a node past an end
        a, b = rng.uniform(-0.5, 0.5, (2, 3)).astype(F)
        c = (a + (b - a) * F(rng.uniform(0.05, 0.95))).astype(F)
        end, other = (a, b) if k % 2 else (b, a)
        lo = (end + (end - other) * F(rng.uniform(0.02, 0.3))).astype(F)
        out.append((np.roll(np.stack([a, b, c]), k // 6, 0), np.append(lo, F(2.0 ** -rng.integers(5, 13)))))
    return out


def want(tri, g4):
    v = [[Fraction(float(x)) for x in p] for p in tri]
    at = [[Fraction(float(g4[a])) + i * Fraction(float(g4[3])) for i in range(N)] for a in range(3)]
    d2 = [squared_distance([x, y, z], *v) for z in at[2] for y in at[1] for x in at[0]]
    return np.sqrt(np.array([float(d) for d in d2])).reshape(N, N, N)


def check(got, tri, g4):
    ref = want(tri, g4)
    # one rounding to FP32, and FP64 steps on coordinates of order 1
    assert np.all(np.abs(np.abs(got.astype(np.float64)) - ref) <= np.spacing(ref.astype(F)) + 32 * 2.0 ** -52)


@pytest.mark.parametrize("case", range(len(slivers())))
def test_point_distance_on_the_host(case):
    from tests.emu import runner
    tri, g4 = slivers()[case]
    check(runner.sdf(tri, np.array([[0, 1, 2]], np.int32), g4, N), tri, g4)


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(slivers())))
def test_build(case):
    import torch
    import paper_2305_07253_amd as hyb
    assert torch.cuda.is_available()
    tri, g4 = slivers()[case]
    sdf = hyb.build_sdf(hyb.build_bvh(tri, np.array([[0, 1, 2]], np.int32)), N, g4)
    check(hyb.sdf_read(sdf).cpu().numpy(), tri, g4)
