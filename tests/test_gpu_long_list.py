"""Lists on either side of the length from which level 1 of the ranking takes
longer sublists (24 000 000 elements): ranks of one list, plain and with sums,
of a few heads, and of a tree's tour."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu

LINE = 24000000


@pytest.mark.parametrize("n", [LINE - 1, LINE, LINE + 4097])
@pytest.mark.parametrize("heads", [1, 3])
def test_list(n, heads):
    g = torch.Generator(device="cuda").manual_seed(n)
    order = torch.randperm(n, device="cuda", generator=g)[: n - n // 50]
    start = (torch.arange(heads, device="cuda") * len(order)) // heads
    nxt = torch.roll(order, -1)
    nxt[(start - 1) % len(order)] = -1
    succ = torch.full((n,), -2, dtype=torch.int32, device="cuda")
    succ[order] = nxt.to(torch.int32)
    at = torch.arange(len(order), device="cuda")
    want = at - start[torch.searchsorted(start, at, right=True) - 1]
    ctx = et.Context()
    head = order[start].to(torch.int32)
    rank = et.et_list_rank(succ, head, ctx=ctx)
    total, again = et.et_list_scan(succ, torch.full_like(succ, 3), head, rank=True, ctx=ctx)
    ctx.check()
    assert torch.equal(rank[order], want.to(torch.int32)) and torch.equal(again, rank)
    assert torch.equal(total[order], (3 * (want + 1)).to(torch.int32))
    assert (rank == -1).sum().item() == n - len(order)
    ctx.close()


@pytest.mark.parametrize("n", [LINE // 2 - 1, LINE // 2])
def test_tree(n):
    parent = gen.random_tree(n, 500, seed=n)
    ref = oracle.euler_tour(parent)
    ctx = et.Context()
    tree = et.et_tree_build(torch.from_numpy(parent).cuda(), ctx=ctx)
    got = tree.export(["rank", "depth", "pre", "size"])
    ctx.check()
    for k in ("rank", "depth", "pre", "size"):
        assert np.array_equal(got[k].cpu().numpy(), ref[k]), k
    tree.free()
    ctx.close()
