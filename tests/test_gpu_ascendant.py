"""The ascendants in both forms (a chain per label below 2^20 nodes, level
by level in ranges of 1024 labels from there on) against the oracle's
top-down definition: tree sizes at the edges of the 256- and 1024-label
ranges and at the line between the forms, on a shallow, a deep and a path
tree."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu
LINE = 1 << 20


@pytest.mark.parametrize("grasp", [None, 300, 1])
@pytest.mark.parametrize("n", [2, 3, 255, 256, 257, 1023, 1025, 4099, LINE - 1, LINE, LINE + 1023, LINE + 1025])
def test_inlabel_tables(n, grasp):
    parent = gen.random_tree(n, grasp, seed=n)
    tour = oracle.euler_tour(parent)
    want = oracle.sv_tables(parent, tour["depth"], tour["pre"], tour["size"])
    tree = et.et_tree_build(torch.from_numpy(parent).cuda())
    got = {k: v.cpu().numpy() for k, v in tree.export(("inlabel", "asc", "depth", "pre", "size")).items()}
    tree.free()
    et.default_context().check()
    for k in ("depth", "pre", "size"):
        assert np.array_equal(got[k], tour[k]), k
    assert np.array_equal(got["inlabel"].view(np.uint32), want["inlabel"].astype(np.uint32))
    assert np.array_equal(got["asc"].view(np.uint32), want["asc"].astype(np.uint32))
