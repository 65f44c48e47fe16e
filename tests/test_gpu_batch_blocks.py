"""Batches at the edges of the batch build's workgroups (4096 nodes): trees
that begin and end with one, cover several, or lie inside one with others;
malformed trees in a workgroup of one tree and of several; and the local walk
of the list ranking at both of its orders (trees of less and of more than 2^19
nodes on average), against the oracle."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu

SIZES = {
    "aligned": [4096, 8192, 4096, 12288], "off_by_one": [4097, 4095, 1, 8191, 3, 4096, 2],
    "mixed": [1, 1, 9000, 5, 4096, 70000, 7, 30, 20000, 1], "one": [40961], "small": [3] * 3000 + [4096],
    "local": [200003, 65536, 300007], "long": [900001, 600001],
}


def _build(parents):
    off = np.concatenate([[0], np.cumsum([len(p) for p in parents])]).astype(np.int64)
    ctx = et.Context()
    tree = et.et_tree_build_batch(torch.from_numpy(np.concatenate(parents)).cuda(), torch.from_numpy(off).cuda(), ctx=ctx)
    return ctx, tree, off


@pytest.mark.parametrize("name", sorted(SIZES))
def test_batch(name):
    parents = [gen.random_tree(n, (None, 7, 1)[i % 3], seed=i) if n > 1 else np.array([-1], dtype=np.int32)
               for i, n in enumerate(SIZES[name])]
    ctx, tree, off = _build(parents)
    got = {k: v.cpu().numpy() for k, v in tree.export().items()}
    rng = np.random.default_rng(1)
    qt = rng.integers(0, len(parents), 5000).astype(np.int32)
    size = np.diff(off)
    qx, qy = ((rng.integers(0, 1 << 40, 5000) % size[qt]).astype(np.int32) for _ in range(2))
    lca = tree.lca_batch(*(torch.from_numpy(a).cuda() for a in (qt, qx, qy))).cpu().numpy()
    ctx.check()
    for t, p in enumerate(parents):
        ref = oracle.euler_tour(p)
        for k in ("depth", "pre", "size"):
            assert np.array_equal(got[k][off[t]:off[t + 1]], ref[k]), (t, k)
        mine = qt == t
        if mine.any():
            assert np.array_equal(lca[mine], oracle.lca_offline(p, qx[mine], qy[mine])), t
    tree.free()
    ctx.close()


@pytest.mark.parametrize("where", [0, 2])
@pytest.mark.parametrize("fault", ["two_roots", "no_root", "self", "range"])
def test_malformed(where, fault):
    parents = [gen.random_tree(n, None, seed=n) for n in (12289, 5000, 50, 60)]
    p = parents[where]
    n = len(p)
    root = int(np.flatnonzero(p == -1)[0])
    other = (root + n // 2) % n
    if fault == "no_root":
        p[root] = other
    else:
        p[other] = {"two_roots": -1, "self": other, "range": n}[fault]
    ctx, tree, _ = _build(parents)
    assert ctx.status_bits() != 0
    tree.free()
    ctx.close()
