"""CPU: the host's tree against a plain sweep over all 32 bins of every axis in FP32
NumPy: the same boxes, splits and leaves, for few and many triangles, triangles whose
centroids coincide along axes, and signed zeros."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
F = np.float32
LEAF_MAX = 4


@pytest.fixture(scope="module")
def builder(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("bvh") / "bvh")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2305_07253_amd", "csrc"),
                    os.path.join(ROOT, "tests", "emu", "bvh.cpp"),
                    os.path.join(ROOT, "paper_2305_07253_amd", "csrc", "bvh_build.cpp"), "-o", exe], check=True)
    return exe


def area(lo, hi):
    e = np.maximum(F(0), hi - lo)
    return F(2) * (e[..., 0] * e[..., 1] + e[..., 1] * e[..., 2] + e[..., 2] * e[..., 0])


def sweep(lo, hi, c, ids, out):
    """Adds (box, depth below, triangles if a leaf) of every node; returns the depth."""
    box = lo[ids].min(0), hi[ids].max(0)
    best = F(np.inf), None
    clo, ext = c[ids].min(0), c[ids].max(0) - c[ids].min(0)
    for a in range(3 if len(ids) > 1 else 0):
        if not ext[a] > 0:
            continue
        b = np.minimum(31, ((c[ids, a] - clo[a]) * (F(32) / ext[a])).astype(np.int32))
        for s in range(31):
            left, right = ids[b <= s], ids[b > s]
            if len(left) and len(right):
                cost = F(1) + F(1) * (area(lo[left].min(0), hi[left].max(0)) * F(len(left)) +
                                      area(lo[right].min(0), hi[right].max(0)) * F(len(right))) / \
                    np.maximum(area(*box), F(1e-30))
                if cost < best[0]:
                    best = cost, (left, right)
    leaf = len(ids) == 1 or (len(ids) <= LEAF_MAX and len(ids) <= best[0])
    out.append((tuple(box[0]) + tuple(box[1]), tuple(sorted(ids)) if leaf else None))
    return 1 if leaf else 1 + max(sweep(lo, hi, c, k, out) for k in best[1])


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 31, 64, 65, 300, 1000])
@pytest.mark.parametrize("kind", ["spread", "flat", "lattice", "zeros"])
def test_tree_is_the_full_sweep(builder, n, kind):
    rng = np.random.default_rng(n)
    c = rng.random((n, 1, 3), dtype=F)
    if kind == "flat":
        c[..., 1] = F(0.5)
    size = F(0.3) if kind == "spread" else F(0.02)
    tri = c + size * (rng.random((n, 3, 3), dtype=F) - F(0.5))
    if kind == "flat":  # centroids coincide along y
        tri[..., 1] = F(0.5) + F(0.25) * np.array([-1, 0, 1], F)
    if kind == "lattice":  # few distinct coordinates, no two triangles alike
        tri = np.round(tri * 16) / F(16)
        tri[:, 0, 0] += np.arange(n, dtype=F) / F(4096)
    if kind == "zeros":
        tri[rng.random(tri.shape) < 0.2] = F(-0.0)
        tri[rng.random(tri.shape) < 0.1] = F(0.0)
    lo, hi = tri.min(1), tri.max(1)
    want = []
    depth = sweep(lo, hi, F(0.5) * (lo + hi), np.arange(n), want)

    raw = subprocess.run([builder], input=tri.astype(F).tobytes(), stdout=subprocess.PIPE, check=True).stdout
    n_nodes, got_depth = np.frombuffer(raw, np.int32, 2)
    nodes = np.frombuffer(raw, F, 16 * n_nodes, 8).reshape(-1, 16)
    slots = np.frombuffer(raw, np.int32, n, 8 + 64 * n_nodes)
    got = []
    for q in nodes:
        ref = q[12:14].view(np.int32)
        for r, x, y, z in ((ref[0], q[0:2], q[2:4], q[8:10]), (ref[1], q[4:6], q[6:8], q[10:12])):
            if x[0] == 1e30:  # the absent child of a tree of one leaf
                continue
            ids = None
            if r < 0:
                first, count = ~r >> 3, ~r & 7
                ids = tuple(sorted(slots[first:first + count]))
            got.append(((x[0], y[0], z[0], x[1], y[1], z[1]), ids))
    inner = [w for w in want if w is not want[0] or w[1] is not None]  # the root's box is stored only if it is a leaf
    assert got_depth == depth
    plain = [sorted((tuple(map(float, box)), ids or ()) for box, ids in x) for x in (got, inner)]
    assert plain[0] == plain[1]
