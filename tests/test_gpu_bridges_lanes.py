"""The one-launch graph batch on 256 lanes a graph (more graphs of at most 256
vertices and 2048 slots than are resident at 1024 lanes) and on either side of
that rule, against the oracle: the largest such graphs, empty ones, one slot
more than the bound, one vertex more, too few graphs, an order, and a
malformed graph among good ones."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


def _graph(n, m, seed):
    if n == 0 or m == 0:
        return np.zeros(n + 1, dtype=np.int32), np.zeros(0, dtype=np.int32)
    return gen.random_multigraph(n, m, seed=seed, loops=False, multi=True)


def _batch(count, big, seed):
    """`count` graphs of up to 256 vertices, some at the bounds, and `big`."""
    rng = np.random.default_rng(seed)
    kinds = [_graph(256, 1024, 1), _graph(256, 300, 2), _graph(0, 0, 0), _graph(7, 0, 0), _graph(1, 0, 0),
             _graph(2, 1, 3), _graph(64, 63, 4), _graph(65, 66, 5), _graph(33, 40, 6), _graph(255, 255, 7), big]
    kinds += [_graph(int(n), int(n * rng.uniform(0.7, 3.0)), i) for i, n in enumerate(rng.integers(3, 257, 40))]
    return kinds, rng.integers(0, len(kinds), count - len(kinds)).tolist()


@pytest.mark.parametrize("count,big", [(2200, (256, 1024)), (2200, (100, 1060)), (2200, (257, 900)), (90, (256, 1024))])
@pytest.mark.parametrize("ordered", [False, True])
def test_lanes(count, big, ordered):
    kinds, rest = _batch(count, _graph(*big, seed=11), count)
    which = list(range(len(kinds))) + rest
    dev = [tuple(torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda() for a in g) for g in kinds]
    want = [oracle.bridges(*g) for g in kinds]
    order = None
    if ordered:
        order = torch.from_numpy(np.random.default_rng(1).permutation(count).astype(np.int32)).cuda()
    ctx = et.Context()
    for _ in range(2):  # the second call finds the counters as the first left them
        mask, spans, counts = et.et_bridges_batch_fused([dev[k] for k in which], ctx=ctx, order=order)
        ctx.check()
        mask, counts = mask.cpu().numpy().view(np.uint32), counts.cpu().numpy()
        for t, k in enumerate(which):
            start, words = spans[t]
            assert counts[t] == want[k][1] and np.array_equal(mask[start:start + words], want[k][0]), (t, k)
    ctx.close()


def test_malformed():
    kinds, rest = _batch(1500, _graph(200, 500, 12), 5)
    row, col = (np.array(a, dtype=np.int32) for a in kinds[0])
    col[5] = 256  # out of range
    kinds[0] = (row, col)
    which = list(range(len(kinds))) + [k for k in rest if k]
    dev = [tuple(torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda() for a in g) for g in kinds]
    want = [oracle.bridges(*g) for g in kinds[1:]]
    ctx = et.Context()
    mask, spans, counts = et.et_bridges_batch_fused([dev[k] for k in which], ctx=ctx)
    assert ctx.status_bits() != 0
    mask, counts = mask.cpu().numpy().view(np.uint32), counts.cpu().numpy()
    assert counts[0] == 0 and not mask[spans[0][0]:spans[0][0] + spans[0][1]].any()
    for t, k in enumerate(which):
        if k:
            start, words = spans[t]
            assert counts[t] == want[k - 1][1] and np.array_equal(mask[start:start + words], want[k - 1][0]), (t, k)
    ctx.close()
