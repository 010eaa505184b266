"""CPU: the stacks of the four-wide tree's traversals hold whatever a tree that the
builder accepts can ask for, also the deepest: clusters that shrink towards a corner, so
that the rest of the tree is always the smallest child and adds a full node's entries."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIMIT = 96
UNSUPPORTED = 4


@pytest.fixture(scope="module")
def stack(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("stack") / "stack")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2305_07253_amd", "csrc"),
                    os.path.join(ROOT, "tests", "emu", "stack.cpp"),
                    os.path.join(ROOT, "paper_2305_07253_amd", "csrc", "bvh_build.cpp"), "-o", exe], check=True)

    def run(tri):
        raw = subprocess.run([exe], input=tri.astype(np.float32).tobytes(), stdout=subprocess.PIPE, check=True).stdout
        return np.frombuffer(raw, np.int32)
    return run


def clusters(levels, last):
    """`levels` clusters of 32 triangles, each a fifth of the one before; `last` at the corner."""
    rng = np.random.default_rng(3)
    out = []
    for k in range(levels):
        at = np.array([1.2, 0.0, 0.0]) + rng.random((32, 1, 3)) * np.array([0.8, 2.0, 2.0])
        out.append(1e4 * 0.2 ** k * (at + 0.02 * (rng.random((32, 3, 3)) - 0.5)))
    at = rng.random((last, 1, 3)) + 0.05 * (rng.random((last, 3, 3)) - 0.5)
    return np.concatenate(out + [1e4 * 0.2 ** levels * at])


def test_deepest_trees(stack):
    bounds, refused = set(), 0
    for levels in range(25, 33):
        for last in range(1, 10):
            rc, bound, most, room = (int(x) for x in stack(clusters(levels, last))[:4])
            if rc == UNSUPPORTED:
                refused += 1
                continue
            assert rc == 0 and bound <= LIMIT
            assert most <= room
            bounds.add(bound)
    assert LIMIT in bounds and refused


@pytest.mark.parametrize("count", [0, 1, 2, 1000])
def test_triangles_stay_where_they_are(stack, count):
    """What the library appends to a tree's triangles moves no megabytes."""
    rc, *_, room = stack(np.random.default_rng(count).random((count, 3, 3)))
    assert rc == 0 and room == 1
