"""The upper levels of the list ranking at list lengths that take each of the
spacing rule's branches: a last level reached by spacing 4 alone, by 8 and
then 4, many heads, few and just over the 1024 that the LDS level takes, and
smaller spacings asked for; ranks and sums of random lists."""
import numpy as np
import pytest
import torch

import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,heads", [
    (50001, 1), (160000, 1), (300000, 1), (600001, 1), (700000, 1), (700000, 1024), (700000, 1025), (1 << 20, 1000),
    (1 << 20, 20000), (3000000, 1), (3000000, 5000), (1 << 22, 3), (9000001, 1),
])
@pytest.mark.parametrize("kn", [3, 1])
def test_levels(n, heads, kn):
    g = torch.Generator(device="cuda").manual_seed(n + heads)
    order = torch.randperm(n, device="cuda", generator=g)[: n - n // 40]
    start = (torch.arange(heads, device="cuda") * len(order)) // heads
    nxt = torch.roll(order, -1)
    nxt[(start - 1) % len(order)] = -1
    succ = torch.full((n,), -2, dtype=torch.int32, device="cuda")
    succ[order] = nxt.to(torch.int32)
    at = torch.arange(len(order), device="cuda")
    want = at - start[torch.searchsorted(start, at, right=True) - 1]
    ctx = et.Context()
    ctx.set_param("lr_kn_log2", kn)
    head = order[start].to(torch.int32)
    rank = et.et_list_rank(succ, head, ctx=ctx)
    total = et.et_list_scan(succ, torch.full_like(succ, -5), head, ctx=ctx)
    ctx.check()
    assert torch.equal(rank[order], want.to(torch.int32))
    assert torch.equal(total[order], (-5 * (want + 1)).to(torch.int32))
    ctx.close()
