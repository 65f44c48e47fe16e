"""The used elements of a weighted ranking, counted while its pairs are made:
either side of the kernel's two shapes and of its largest grid, lists with
unused slots, and a list that one used element is not on."""
import numpy as np
import pytest
import torch

import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1025, 20001, (1 << 18) - 1, 1 << 18, (1 << 18) + 4097, (1 << 22) + 1, 5000001])
@pytest.mark.parametrize("stray", [False, True])
def test_scan(n, stray):
    rng = np.random.default_rng(n)
    order = rng.permutation(n)[: n - n // 9]
    succ = np.full(n, -2, dtype=np.int32)
    succ[order[:-1]] = order[1:]
    succ[order[-1]] = -1
    weight = rng.integers(-1000, 1000, n).astype(np.int32)
    if stray:
        unused = np.flatnonzero(succ == -2)
        succ[unused[len(unused) // 2]] = -1  # a used element that no head leads to
    ctx = et.Context()
    head = torch.from_numpy(order[:1].astype(np.int32)).cuda()
    total, rank = et.et_list_scan(torch.from_numpy(succ).cuda(), torch.from_numpy(weight).cuda(), head, rank=True, ctx=ctx)
    if stray:
        assert ctx.status_bits() != 0
    else:
        ctx.check()
        rank, total = rank.cpu().numpy(), total.cpu().numpy()
        assert np.array_equal(rank[order], np.arange(len(order)))
        assert np.array_equal(total[order], np.cumsum(weight[order], dtype=np.int64).astype(np.int32))
    ctx.close()
