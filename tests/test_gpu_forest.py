"""The spanning forest of the bridge call (first round without atomics,
linked half-edge lists, component chaining) on the shapes where it can go
wrong, against the oracle: local minima, hubs with the smallest and the
largest id, self-loops and parallel edges in a row's first slots, isolated
vertices, and many components around the 4096 vertices that one workgroup of
the root pass takes."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


def _pairs(n):
    """n // 2 components of two vertices; an odd last vertex stays isolated."""
    a = np.arange(0, n - 1, 2)
    return gen.csr_from_pairs(n, a, a + 1)


def _hub(n, hub):
    """A hub joined to every vertex, and every third leaf to the next one."""
    leaves = np.delete(np.arange(n), hub)
    third = leaves[:-1:3]
    nxt = leaves[1::3][: len(third)]
    return gen.csr_from_pairs(n, np.concatenate([np.full(n - 1, hub), third]), np.concatenate([leaves, nxt]))


def _first_slots(n, seed):
    """Self-loops and parallel copies on a path with chords, isolated vertices at the end."""
    rng = np.random.default_rng(seed)
    m = n - 5
    a = np.arange(m - 1)
    loops = rng.integers(0, m, m // 4)
    twice = a[rng.random(m - 1) < 0.3]
    chord = rng.integers(0, m, (2, m // 16))
    u = np.concatenate([a, loops, twice, chord[0]])
    w = np.concatenate([a + 1, loops, twice + 1, chord[1]])
    return gen.csr_from_pairs(n, u, w)


def _zigzag(n):
    """A path through small and large ids in turn: every second vertex is a local minimum."""
    order = np.empty(n, dtype=np.int64)
    order[::2] = np.arange((n + 1) // 2)
    order[1::2] = np.arange((n + 1) // 2, n)
    return gen.csr_from_pairs(n, order[:-1], order[1:])


GRAPHS = {
    "pairs_4095": lambda: _pairs(4095), "pairs_4096": lambda: _pairs(4096), "pairs_4097": lambda: _pairs(4097),
    "pairs_20001": lambda: _pairs(20001),
    "hub_first": lambda: _hub(5000, 0), "hub_last": lambda: _hub(5000, 4999), "hub_middle": lambda: _hub(777, 300),
    "first_slots": lambda: _first_slots(3001, 1), "first_slots_small": lambda: _first_slots(37, 2),
    "zigzag": lambda: _zigzag(4099), "two": lambda: gen.csr_from_pairs(2, [0], [1]),
    "loop_only": lambda: gen.csr_from_pairs(3, [1], [1]),
    "random": lambda: gen.random_multigraph(4097, 6000, seed=3),
    # both sides of the sampling rule, and block counts at the sparse table's steps
    "sparse_66000": lambda: gen.random_multigraph(66000, 150000, seed=4),
    "dense_66000": lambda: gen.random_multigraph(66000, 400000, seed=5),
    "slots_2to14": lambda: gen.random_multigraph(3000, 1 << 13, seed=6),
    "slots_more": lambda: gen.random_multigraph(3000, (1 << 13) + 1, seed=7),
    "blocks_64": lambda: gen.random_multigraph(2048, 2300, seed=8),
    "blocks_129": lambda: gen.random_multigraph(4100, 5000, seed=9),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_forest_shapes(name):
    row, col = GRAPHS[name]()
    d = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda() for a in (row, col)]
    want, count = oracle.bridges(row, col)
    ctx = et.Context()
    for call in (lambda: et.et_bridges(*d, ctx=ctx), lambda: et.et_bridges_ck(*d, spanning="forest", ctx=ctx),
                 lambda: et.et_bridges_ck(*d, spanning="bfs", ctx=ctx)):
        mask, got = call()
        ctx.check()
        assert got == count
        assert np.array_equal(mask.cpu().numpy().view(np.uint32)[: len(want)], want)
    ctx.close()
