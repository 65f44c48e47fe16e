"""Radix passes of every digit width (7 to 11 bits) on both sides of the lines
between their numbers, against the oracle's successors: trees whose parents
spread over all digits, lie in one digit, and ascend; and edge lists, whose
half-edges are sorted by target and by source."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu

SHAPES = {"random": lambda n: gen.random_tree(n, None, seed=n), "near": lambda n: gen.random_tree(n, 5, seed=n),
          "star": lambda n: gen.star_tree(n, root=n // 3), "path": lambda n: gen.path_tree(n, seed=n)}


@pytest.mark.parametrize("n,shape", [
    (4097, "random"), (65536, "near"), (65537, "random"), (131072, "star"), (131073, "path"), (262144, "random"),
    (262145, "random"), (300007, "star"), (524289, "near"), (1 << 20, "random"), ((1 << 20) + 1, "random"),
    ((1 << 20) + 4097, "path"), ((1 << 21) - 1, "star"), (1 << 21, "random"), ((1 << 21) + 1, "random"),
    ((1 << 24) + 1, "near"),
])
def test_tree(n, shape):
    parent = SHAPES[shape](n)
    succ, _ = oracle.tree_succ(parent)
    ctx = et.Context()
    tree = et.et_tree_build(torch.from_numpy(parent).cuda(), ctx=ctx)
    got = tree.export()["succ"].cpu().numpy()
    ctx.check()
    assert np.array_equal(got, succ)
    tree.free()
    ctx.close()


@pytest.mark.parametrize("n", [3000, 131073, 262145, 500001, (1 << 20) + 1, (1 << 20) + 2])
def test_edges(n):
    parent = gen.random_tree(n, None, seed=n)
    child = np.flatnonzero(parent >= 0)
    rng = np.random.default_rng(n)
    flip = rng.random(len(child)) < 0.5
    order = rng.permutation(len(child))
    u = np.where(flip, child, parent[child])[order].astype(np.int32)
    v = np.where(flip, parent[child], child)[order].astype(np.int32)
    root = int(np.flatnonzero(parent == -1)[0])
    want = oracle.euler_tour_edges(n, u, v, root)
    ctx = et.Context()
    tree = et.et_tree_build_edges(torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda(), n, root, ctx=ctx)
    got = {k: a.cpu().numpy() for k, a in tree.export().items()}
    ctx.check()
    for k in ("succ", "rank"):
        assert np.array_equal(got[k][: 2 * (n - 1)], want[k]), k
    for k in ("depth", "pre", "size"):
        assert np.array_equal(got[k], want[k]), k
    tree.free()
    ctx.close()
