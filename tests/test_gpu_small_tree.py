"""The one-launch build of a small tree against the oracle: every table it
leaves behind (tour, ranks, statistics, Inlabel tables through export and
queries), at the edges of its sizes, of its wavefronts and of its sublist
spacings, on either side of the line to the multi-kernel build; malformed
parent arrays; and the calls that go on from its tables."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


def _d(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


SHAPES = {
    "random": lambda n: gen.random_tree(n, None, seed=n), "deep": lambda n: gen.random_tree(n, 9, seed=n),
    "path": lambda n: gen.path_tree(n, seed=n), "star": lambda n: gen.star_tree(n, root=n // 2),
}


@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 511, 513, 1024, 1025, 2049, 4095, 4096, 4097])
def test_tables(n, shape):
    parent = SHAPES[shape](n)
    ref = oracle.euler_tour(parent)
    tab = oracle.sv_tables(parent, ref["depth"], ref["pre"], ref["size"])
    succ, _ = oracle.tree_succ(parent)
    qx, qy = gen.random_queries(n, 3000, seed=n)
    ctx = et.Context()
    tree = et.et_tree_build(_d(parent), ctx=ctx)
    got = {k: v.cpu().numpy() for k, v in tree.export().items()}
    tour = tree.tour().cpu().numpy()
    lca = tree.lca(_d(qx), _d(qy)).cpu().numpy()
    rmq = tree.rmq_build(_d(parent)).lca_rmq(_d(qx), _d(qy)).cpu().numpy()
    ctx.check()
    assert np.array_equal(got["succ"], succ)
    for k in ("rank", "depth", "pre", "size"):
        assert np.array_equal(got[k], ref[k]), k
    assert np.array_equal(got["inlabel"].view(np.uint32), tab["inlabel"])
    assert np.array_equal(got["asc"].view(np.uint32), tab["asc"])
    want = np.empty(2 * (n - 1), dtype=np.int32)
    on = np.flatnonzero(ref["rank"] >= 0)
    want[ref["rank"][on]] = on
    assert np.array_equal(tour, want)
    answers = oracle.lca_offline(parent, qx, qy)
    assert np.array_equal(lca, answers) and np.array_equal(rmq, answers)
    tree.free()
    ctx.close()


@pytest.mark.parametrize("n", [2, 65, 1500, 4096])
@pytest.mark.parametrize("fault", ["no_root", "two_roots", "self", "range", "cycle"])
def test_malformed(n, fault):
    parent = gen.random_tree(n, None, seed=3)
    root = int(np.flatnonzero(parent == -1)[0])
    other = (root + 1) % n
    if fault == "no_root":
        parent[root] = other
    elif fault == "two_roots":
        parent[other] = -1
    elif fault == "self":
        parent[other] = other
    elif fault == "range":
        parent[other] = n
    else:  # two nodes above each other (with two nodes: no root is left)
        a, b = other, (root + 2) % n if n > 2 else root
        parent[a], parent[b] = b, a
    ctx = et.Context()
    tree = et.et_tree_build(_d(parent), ctx=ctx)
    assert ctx.status_bits() != 0
    qx, qy = gen.random_queries(n, 100, seed=1)
    tree.lca(_d(qx), _d(qy))  # unspecified answers, but no fault
    tree.export()
    ctx.status_bits()
    tree.free()
    ctx.close()
