"""Graphs whose ids follow their shape (cycles, strips, neighbours by id): the
trees of the first hooking round are chains as long as the graph there. Bridges
against the oracle, and the time of the call against that of the same graph
with its ids shuffled: climbing such chains link by link takes 50 to 300 times
as long, compressed ones at most 5 times."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


def _pairs(kind, n):
    i = np.arange(n, dtype=np.int64)
    if kind == "cycle":
        return i, (i + 1) % n
    if kind == "strip":  # a band of triangles
        return np.concatenate([i[:-2], i[:-1]]), np.concatenate([i[2:], i[1:]])
    if kind == "near":
        d = np.random.default_rng(n).integers(1, 40, (3, n))
        return np.tile(i, 3), ((i + d) % n).ravel()
    if kind == "path":
        return i[:-1], i[1:]
    # a cycle whose ids alternate between its halves: every second vertex is a
    # local minimum, and these form a chain of their own
    u, v = _pairs("cycle", n)
    at = np.where(i % 2 == 0, i // 2, (n + 1) // 2 + i // 2)
    return at[u], at[v]


def _csr(u, v, n):
    key = np.sort(np.concatenate([u * n + v, v * n + u]))
    rp = np.zeros(n + 1, dtype=np.int64)
    rp[1:] = np.cumsum(np.bincount(key // n, minlength=n))
    return rp.astype(np.int32), (key % n).astype(np.int32)


def _run(rp, col):
    rp, col = torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda()
    times = []
    for _ in range(6):
        torch.cuda.synchronize()
        t = time.perf_counter()
        mask, count = et.et_bridges(rp, col)
        times.append(time.perf_counter() - t)
    et.default_context().check()
    return mask.cpu().numpy().view(np.uint32), count, sorted(times)[2]


@pytest.mark.parametrize("kind", ["cycle", "strip", "near", "path", "halves"])
@pytest.mark.parametrize("n", [2, 3, 900, 4096, 4097, 100000, 400000, 600000])
def test_ids_that_follow_the_shape(kind, n):
    u, v = _pairs(kind, n)
    keep = u != v
    u, v = u[keep], v[keep]
    rp, col = _csr(u, v, n)
    mask, count, t = _run(rp, col)
    want, want_count = oracle.bridges(rp, col)
    assert count == want_count and np.array_equal(mask[: len(want)], want)
    if n >= 100000:
        p = np.random.default_rng(n).permutation(n)
        assert t < 12 * _run(*_csr(p[u], p[v], n))[2]


@pytest.mark.parametrize("kind", ["halves", "near", "shaken"])
def test_pick_samples_compressed_trees(kind):
    """Above 2^20 vertices, where labels follow the pick: its 1024 samples are
    one gather each (20 us), not a climb of the second round's chains."""
    n = (1 << 21) + 5
    if kind == "shaken":  # a strip with its ids exchanged within short distances
        u, v = _pairs("strip", n)
        at = np.empty(n, dtype=np.int64)
        at[np.argsort(np.arange(n) + 64 * np.random.default_rng(7).random(n))] = np.arange(n)
        u, v = at[u], at[v]
    else:
        u, v = _pairs(kind, n)
    rp, col = _csr(u, v, n)
    ctx = et.Context()
    d = [torch.from_numpy(a).cuda() for a in (rp, col)]
    et.et_bridges(*d, ctx=ctx)
    ctx.profile(True, only="k_big_component")
    for _ in range(3):
        mask, count = et.et_bridges(*d, ctx=ctx)
    launches, total, _ = ctx.profile_read()["k_big_component"]
    ctx.check()
    ctx.close()
    want, want_count = oracle.bridges(rp, col)
    assert count == want_count and np.array_equal(mask.cpu().numpy().view(np.uint32)[: len(want)], want)
    assert total / launches < 0.08
