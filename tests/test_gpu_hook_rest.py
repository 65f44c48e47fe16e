"""The last hooking phase of the spanning forest on sampled graphs, with byte
labels (more than 2^20 vertices) and without: numbers of components below,
at and above what the labels hold, components joined only by slots that the
samples leave out, one component that holds nearly all vertices, rows longer
than a workgroup's pass, and malformed rows; against the oracle."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu

LINE = 1 << 20


def _blobs(n, k, degree, joins, seed, share=0.0):
    """k random blobs over a shuffled vertex set (the first one holds `share`
    of the vertices on top of its part), and `joins` edges between random
    vertices of any two."""
    rng = np.random.default_rng(seed)
    blob = np.where(rng.random(n) < share, 0, rng.integers(0, k, n))
    order = np.argsort(blob, kind="stable")
    size = np.bincount(blob, minlength=k)
    lo = np.cumsum(size) - size
    u = rng.integers(0, n, n * degree // 2)
    w = order[lo[blob[u]] + rng.integers(0, 1 << 40, len(u)) % size[blob[u]]]
    x = rng.integers(0, n, (2, joins))
    return gen.csr_from_pairs(n, np.concatenate([u, x[0]]), np.concatenate([w, x[1]]))


def _hub(n):
    rng = np.random.default_rng(n)
    far = rng.choice(n - 1, n // 4, replace=False)  # all of the last vertex's row
    u = rng.integers(0, n, n)
    return gen.csr_from_pairs(n, np.concatenate([u, far]), np.concatenate([(u + 1) % n, np.full(len(far), n - 1)]))


GRAPHS = {
    "line_few": lambda: _blobs(LINE, 7, 10, 3, 1), "above_few": lambda: _blobs(LINE + 1, 7, 10, 3, 2),
    "one": lambda: _blobs(LINE + 300, 1, 16, 0, 3), "fit": lambda: _blobs(LINE + 511, 200, 12, 150, 4),
    "full": lambda: _blobs(LINE + 77, 256, 12, 40, 5), "too_many": lambda: _blobs(LINE + 5, 1500, 10, 900, 6),
    "half_named": lambda: _blobs(LINE + 9, 600, 12, 100, 7, share=0.5),
    "mostly_one": lambda: _blobs(LINE + 9, 400, 12, 100, 8, share=0.97),
    "sparse": lambda: _blobs(LINE + 4099, 50, 3, 30, 9), "hub": lambda: _hub(LINE + 259),
    "unlabelled": lambda: _blobs(70001, 300, 10, 100, 10), "unlabelled_small": lambda: _blobs(6001, 9, 12, 4, 11),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_hook_rest(name):
    row, col = GRAPHS[name]()
    d = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda() for a in (row, col)]
    want, count = oracle.bridges(row, col)
    ctx = et.Context()
    for call in (lambda: et.et_bridges(*d, ctx=ctx), lambda: et.et_bridges_ck(*d, spanning="forest", ctx=ctx)):
        mask, got = call()
        ctx.check()
        assert got == count
        assert np.array_equal(mask.cpu().numpy().view(np.uint32)[: len(want)], want)
    ctx.close()


@pytest.mark.parametrize("fault", ["column", "rows"])
def test_malformed(fault):
    row, col = (np.array(a, dtype=np.int32) for a in _blobs(LINE + 300, 40, 10, 3, 12))
    n = len(row) - 1
    if fault == "column":
        col[row[n // 2 + 1] - 1] = n
    else:
        row[n // 2] = row[n // 2 + 9]
    ctx = et.Context()
    et.et_bridges(*[torch.from_numpy(a).cuda() for a in (row, col)], ctx=ctx)
    assert ctx.status_bits() != 0
    ctx.close()
