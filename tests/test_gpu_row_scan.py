"""The neighbour extremes of the bridge call against the oracle: rows that
several lanes share (dense graphs), workgroups whose rows exceed the LDS
stage, rows longer than a workgroup, and vertex counts on both sides of the
lines where the gathers take another pass over the columns (1.5 * 2^20
vertices a pass, at least six slots a vertex)."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu
PASS = 3 << 19


def _graph(n, degree, hubs, seed):
    """Random pairs, a few hubs joined to spread-out vertices, and a tail of bridges hung on vertex 0."""
    rng = np.random.default_rng(seed)
    m = n * degree // 2
    core = n - n // 50  # the other vertices make a path
    u, w = rng.integers(0, core, m), rng.integers(0, core, m)
    parts_u, parts_w = [u], [w]
    for h in range(hubs):
        spokes = rng.choice(core, size=min(core - 1, 7000 + 500 * h), replace=False)
        parts_u.append(np.full(spokes.shape[0], rng.integers(0, core)))
        parts_w.append(spokes)
    path = np.concatenate([[0], np.arange(core, n)])
    parts_u.append(path[:-1])
    parts_w.append(path[1:])
    perm = rng.permutation(n)
    return gen.csr_from_pairs(n, perm[np.concatenate(parts_u)], perm[np.concatenate(parts_w)])


@pytest.mark.parametrize("n,degree,hubs", [
    (300, 100, 0), (1000, 40, 0), (1001, 24, 0), (4000, 300, 0),  # 2 .. 16 lanes a row; rows above 512 slots
    (20000, 3, 3), (20000, 17, 2), (255, 16, 1), (257, 16, 1),    # hubs beyond the stage; row-block edges
    (PASS - 1, 7, 2), (PASS, 7, 1), (PASS + 1, 7, 2), (2 * PASS + 3, 7, 1), (2 * PASS + 3, 4, 1),
])
def test_row_scan(n, degree, hubs):
    row, col = _graph(n, degree, hubs, seed=n + degree)
    want, count = oracle.bridges(row, col)
    mask, got = et.et_bridges(*(torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda() for a in (row, col)))
    et.default_context().check()
    assert got == count
    assert np.array_equal(mask.cpu().numpy().view(np.uint32)[: len(want)], want)
