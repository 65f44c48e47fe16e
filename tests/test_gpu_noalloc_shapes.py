"""et_list_rank_noalloc takes every list within its limits at every launch
shape: the longest list with numbers of heads up to the most, where the levels
above the first one shrink least and need the most scratch (44 466 528 bytes at
52437 heads with "lr_k1_log2" 1 and "lr_kn_log2" 2)."""
import pytest
import torch

import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k1,kn", [(1, 1), (1, 2), (1, 3), (1, 4), (1, 10), (2, 2), (4, 3), (10, 10)])
def test_longest_list(k1, kn):
    n = et.et.NOALLOC_MAX_LEN
    ctx = et.Context()
    ctx.set_param("lr_k1_log2", k1)
    ctx.set_param("lr_kn_log2", kn)
    order = torch.randperm(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(k1 * 16 + kn))
    rank = torch.empty(n, dtype=torch.int32, device="cuda")
    for heads in [1, 1024, 1025, 46267, 49000, 52217, 52381, 52437, 52500, 56000, 60000, et.et.NOALLOC_MAX_HEADS]:
        start = (torch.arange(heads, device="cuda") * n) // heads
        nxt = torch.roll(order, -1)
        nxt[start - 1] = -1
        succ = torch.empty(n, dtype=torch.int32, device="cuda")
        succ[order] = nxt.to(torch.int32)
        et.et.et_list_rank_noalloc(succ, order[start].to(torch.int32), rank, ctx=ctx)
        at = torch.arange(n, device="cuda")
        want = at - start[torch.searchsorted(start, at, right=True) - 1]
        assert torch.equal(rank[order].long(), want), heads
    ctx.check()
    ctx.close()
