"""Small trees of regular ids: `legs` paths below the root, each of every
legs-th id, so that ids of one residue lie one after the other on the tour. One
tree and a batch in one launch against the oracle, and their times against
those of paths in id order: sublists that start at regular ids take 20 to 35
times as long, pseudo-random ones less than 3 times."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


def _d(a, t=np.int32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=t)).cuda()


def _legs(n, legs):
    parent = np.maximum(np.arange(n) - legs, 0)
    parent[0] = -1
    return parent.astype(np.int32)


def _median(call):
    times = []
    for _ in range(9):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(8):
            call()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    return sorted(times)[4]


@pytest.mark.parametrize("n", [5, 600, 1024, 1025, 2048, 3000, 4095, 4096])
@pytest.mark.parametrize("legs", [1, 2, 3, 8, 64, 511])
def test_tables(n, legs):
    parent = _legs(n, legs)
    ref = oracle.euler_tour(parent)
    succ, _ = oracle.tree_succ(parent)
    rng = np.random.default_rng(n)
    qx, qy = rng.integers(0, n, (2, 500)).astype(np.int32)
    ctx = et.Context()
    tree = et.et_tree_build(_d(parent), ctx=ctx)
    got = {k: v.cpu().numpy() for k, v in tree.export().items()}
    lca = tree.lca(_d(qx), _d(qy)).cpu().numpy()
    off, qoff = _d([0, n], np.int64), _d([0, 500], np.int64)
    out = et.et_lca_batch_fused(_d(parent), off, qoff, _d(qx), _d(qy), n, ctx=ctx).cpu().numpy()
    ctx.check()
    tree.free()
    ctx.close()
    assert np.array_equal(got["succ"], succ)
    for k in ("rank", "depth", "pre", "size"):
        assert np.array_equal(got[k], ref[k]), k
    want = oracle.lca_offline(parent, qx, qy)
    assert np.array_equal(lca, want) and np.array_equal(out, want)


def test_times():
    n, trees = 4096, 600
    off, qoff = _d(np.arange(trees + 1) * n, np.int64), _d(np.arange(trees + 1) * 4, np.int64)
    qx = torch.ones(4 * trees, dtype=torch.int32, device="cuda")
    qy = torch.full_like(qx, n - 1)

    def both(legs):
        one = _d(_legs(n, legs))
        many = one.repeat(trees)
        return (_median(lambda: et.et_tree_build(one).free()),
                _median(lambda: et.et_lca_batch_fused(many, off, qoff, qx, qy, n)))

    path, path_batch = both(1)
    for legs in (8, 16):
        one, batch = both(legs)
        assert one < 5 * path and batch < 5 * path_batch, legs
