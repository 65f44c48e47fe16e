"""Successors stored in two passes (one tree of at least 12 000 000 nodes)
against the oracle's: either side of the line, ragged and whole tiles and
ranges of children, shapes whose children fall into one range at a time and
into all at once, the size from which a range holds 131072 children, a root
at either end of the grouped order, and malformed parent arrays."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu

LINE = 12000000


@pytest.mark.parametrize("n,shape", [
    (LINE - 1, "random"), (LINE, "random"), (LINE, "star"), (LINE + 1, "path"), (184 << 16, "relabel"),
    ((184 << 16) + 1, "random"), ((1 << 25) - 1, "path"), ((1 << 25) + 5, "star"),
])
def test_successors(n, shape):
    parent = {"random": lambda: gen.random_tree(n, None, seed=1), "star": lambda: gen.star_tree(n, root=n - 1),
              "path": lambda: gen.path_tree(n), "relabel": lambda: gen.path_tree(n, seed=2)}[shape]()
    succ, _ = oracle.tree_succ(parent)
    ctx = et.Context()
    tree = et.et_tree_build(torch.from_numpy(parent).cuda(), ctx=ctx)
    got = tree.export()["succ"].cpu().numpy()
    ctx.check()
    assert np.array_equal(got, succ)
    tree.free()
    ctx.close()


@pytest.mark.parametrize("fault", ["two_roots", "self", "range"])
def test_malformed(fault):
    n = LINE + 3
    parent = gen.path_tree(n)
    other = int(np.flatnonzero(parent != -1)[n // 2])
    parent[other] = {"two_roots": -1, "self": other, "range": n}[fault]
    ctx = et.Context()
    tree = et.et_tree_build(torch.from_numpy(parent).cuda(), ctx=ctx)
    assert ctx.status_bits() != 0
    tree.free()
    ctx.close()
