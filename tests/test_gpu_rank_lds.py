"""Lists that one workgroup ranks in LDS, whole (up to 8192 elements and
1024 heads) or as the last level (up to 12288) of a longer list, against the oracle: sizes
on both sides of those lines and of the chunk spacings, orders in which one
sublist is very long, weighted scans that wrap, and malformed lists."""
import numpy as np
import pytest
import torch

import oracle
import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


def _d(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _lists(order, nlists, L, rng):
    cuts = np.sort(rng.choice(np.arange(1, len(order)), nlists - 1, replace=False)) if nlists > 1 else []
    succ = np.full(L, -2, dtype=np.int32)
    heads = []
    for part in np.split(order, cuts):
        succ[part[:-1]] = part[1:]
        succ[part[-1]] = -1
        heads.append(part[0])
    return succ, np.array(heads, dtype=np.int32)


def _check(succ, heads, rng):
    w = rng.integers(-(1 << 31), 1 << 31, len(succ)).astype(np.int32)
    ctx = et.default_context()
    rank = et.et_list_rank(_d(succ), _d(heads)).cpu().numpy()
    total, rank2 = et.et_list_scan(_d(succ), _d(w), _d(heads), rank=True)
    only = et.et_list_scan(_d(succ), _d(w), _d(heads)).cpu().numpy()
    ctx.check()
    want = oracle.list_rank(succ, heads)
    sums = oracle.list_scan(succ, w, heads)
    sums = sums[0] if isinstance(sums, tuple) else sums
    assert np.array_equal(rank, want) and np.array_equal(rank2.cpu().numpy(), want)
    assert np.array_equal(total.cpu().numpy(), sums) and np.array_equal(only, sums)


@pytest.mark.parametrize("L", [1, 2, 63, 1023, 1024, 1025, 2048, 2049, 8191, 8192, 8193, 12289, 48700, 48900,
                               200003])
@pytest.mark.parametrize("nlists", [1, 9, 1023, 1024, 1025, 3000])
def test_sizes(L, nlists):
    rng = np.random.default_rng(L * 5000 + nlists)
    order = rng.permutation(L)[: max(1, L - L // 7)]
    _check(*_lists(order, min(nlists, len(order)), L, rng), rng)


@pytest.mark.parametrize("L", [4096, 8192])
@pytest.mark.parametrize("stride", [1, 4, 16, 1024, -1])
def test_orders(L, stride):
    if stride > 0:  # all ids of one residue after another
        order = np.concatenate([np.arange(r, L, stride) for r in range(stride)])
    else:
        order = np.arange(L - 1, -1, -1)
    rng = np.random.default_rng(L + stride)
    _check(*_lists(order, 1, L, rng), rng)


@pytest.mark.parametrize("L", [40, 1500, 8000])
@pytest.mark.parametrize("fault", ["cycle", "shared", "range", "unused", "head_twice", "head_inside", "no_head"])
def test_malformed(L, fault):
    rng = np.random.default_rng(L)
    order = rng.permutation(L)[: L - 5]
    succ, heads = _lists(order, 3, L, rng)
    unused = np.flatnonzero(succ == -2)
    at = order[L // 2]
    if fault == "cycle":
        succ[order[-1]] = order[-4]
    elif fault == "shared":
        succ[at] = order[3] if order[3] not in heads else order[4]
    elif fault == "range":
        succ[at] = L + 7
    elif fault == "unused":
        succ[at] = unused[0]
    elif fault == "head_twice":
        heads = np.concatenate([heads, heads[:1]])
    elif fault == "head_inside":
        inside = next(e for e in order[2:] if e not in heads)
        heads = np.concatenate([heads, [inside]])
    else:
        heads = heads[:-1]
    et.et_list_rank(_d(succ), _d(heads))
    assert et.default_context().status_bits() != 0
