"""Lists on either side of the length from which level 1 of the ranking takes
longer sublists and fewer of them a wavefront (2^25 elements): ranks and sums
of one list and of a few, in id order, against it and shuffled, a tree's tour,
and the time of the level-1 walk on a list in id order against a shuffled
one's: 0.8 with 256 sublists a wavefront, 0.63 with 64."""
import pytest
import torch

import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu

LINE = 1 << 25


def _order(n, kind):
    if kind == "shuffled":
        return torch.randperm(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    i = torch.arange(n, device="cuda")
    return i if kind == "forward" else i.flip(0)


def _list(order, n, heads):
    start = (torch.arange(heads, device="cuda") * len(order)) // heads
    nxt = torch.roll(order, -1)
    nxt[(start - 1) % len(order)] = -1
    succ = torch.full((n,), -2, dtype=torch.int32, device="cuda")
    succ[order] = nxt.to(torch.int32)
    return succ, order[start].to(torch.int32), start


@pytest.mark.parametrize("n", [LINE - 1, LINE, LINE + 4097])
@pytest.mark.parametrize("heads", [1, 3])
@pytest.mark.parametrize("kind", ["forward", "backward", "shuffled"])
def test_list(n, heads, kind):
    order = _order(n, kind)[: n - n // 50]
    succ, head, start = _list(order, n, heads)
    at = torch.arange(len(order), device="cuda")
    want = (at - start[torch.searchsorted(start, at, right=True) - 1]).to(torch.int32)
    ctx = et.Context()
    rank = et.et_list_rank(succ, head, ctx=ctx)
    total, again = et.et_list_scan(succ, torch.full_like(succ, 3), head, rank=True, ctx=ctx)
    ctx.check()
    assert torch.equal(rank[order], want) and torch.equal(again, rank)
    assert torch.equal(total[order], 3 * (want + 1))
    assert (rank == -1).sum().item() == n - len(order)
    ctx.close()


@pytest.mark.parametrize("n", [LINE // 2 - 1, LINE // 2, LINE // 2 + 70001])
@pytest.mark.parametrize("legs", [1, 64, 0])
def test_tour(n, legs):
    i = torch.arange(n, device="cuda")
    if legs:
        parent = (i - legs).clamp(min=0)
    else:
        g = torch.Generator(device="cuda").manual_seed(n)
        parent = (torch.rand(n, device="cuda", generator=g, dtype=torch.float64) * i).long()
    parent[0] = -1
    ctx = et.Context()
    tree = et.et_tree_build(parent.int(), ctx=ctx)
    got = tree.export(["succ", "rank", "depth"])
    ctx.check()
    rank, succ = got["rank"].long(), got["succ"].long()
    tour = torch.arange(2 * n, device="cuda")[2:]
    assert rank[:2].tolist() == [-1, -1]
    assert torch.equal(rank[tour].sort().values, torch.arange(2 * n - 2, device="cuda"))
    on = tour[succ[tour] >= 0]
    assert len(on) == 2 * n - 3 and torch.equal(rank[succ[on]], rank[on] + 1)
    depth = got["depth"].long()
    assert depth[0] == 0 and torch.equal(depth[1:], depth[parent[1:]] + 1)
    tree.free()
    ctx.close()


def test_times():
    ms = []
    for kind in ("forward", "shuffled"):
        succ, head, _ = _list(_order(LINE, kind), LINE, 1)
        ctx = et.Context()
        rank = torch.empty_like(succ)
        et.et_list_rank(succ, head, rank, ctx=ctx)
        ctx.profile(True, only="k_walk1<false>")
        for _ in range(5):
            et.et_list_rank(succ, head, rank, ctx=ctx)
        launches, total, _ = ctx.profile_read()["k_walk1<false>"]
        ms.append(total / launches)
        ctx.check()
        ctx.close()
    assert ms[0] < 0.72 * ms[1], ms
