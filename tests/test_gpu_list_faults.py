"""Malformed lists whose every element is still walked from a head, so that
only the fault itself can give them away: each one sets a status bit, in a
plain ranking and in a weighted scan, at sizes of every form of the last level
(one workgroup's LDS with every element or some of them starting a sublist,
upper levels, more heads than the LDS form takes)."""
import numpy as np
import pytest
import torch

import paper_2103_15217_amd as et

pytestmark = pytest.mark.gpu


def _d(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _flagged(succ, heads):
    ctx = et.default_context()
    s, h = _d(succ), _d(heads)
    et.et_list_rank(s, h)
    plain = ctx.status_bits()
    et.et_list_scan(s, torch.ones_like(s), h)
    return plain != 0 and ctx.status_bits() != 0


def _chain(order, nlists, L):
    """`order` cut into nlists lists of even length in L slots."""
    succ = np.full(L, -2, dtype=np.int32)
    parts = np.array_split(order, nlists)
    for part in parts:
        succ[part[:-1]] = part[1:]
        succ[part[-1]] = -1
    return succ, np.array([part[0] for part in parts], dtype=np.int32), parts


SIZES = [(6, 1), (40, 3), (1000, 1), (1025, 7), (1500, 700), (2048, 1), (2049, 2), (5000, 1000), (8192, 1),
         (8193, 1), (9000, 2000), (30000, 3), (30000, 12000), (100000, 20000)]


@pytest.mark.parametrize("L,nlists", SIZES)
def test_last_element_names_an_unused_slot(L, nlists):
    rng = np.random.default_rng(L + nlists)
    succ, heads, parts = _chain(rng.permutation(L)[: L - max(1, L // 9)], nlists, L)
    unused = np.flatnonzero(succ == -2)
    for slot in unused[rng.permutation(len(unused))[:12]]:
        bad = succ.copy()
        bad[parts[rng.integers(len(parts))][-1]] = slot
        assert _flagged(bad, heads), (L, nlists, int(slot))


@pytest.mark.parametrize("L", [40, 1025, 3000, 8000, 8193, 30000])
def test_one_element_list_named_twice(L):
    rng = np.random.default_rng(L)
    for gap in (1, 64, 65, 300):  # lanes of one wavefront, of two, of two workgroup rounds
        for _ in range(6):
            order = rng.permutation(L)
            succ = np.full(L, -2, dtype=np.int32)
            n = min(L // 2, 900)
            succ[order[:n]] = -1
            heads = order[:n].astype(np.int32)
            at = int(rng.integers(0, n))
            assert _flagged(succ, np.insert(heads, min(n, at + gap), heads[at])), (L, gap, at)


@pytest.mark.parametrize("L", [40, 1025, 3000, 8000, 8193, 30000])
@pytest.mark.parametrize("depth", [1, 2, 5])
def test_two_heads_share_a_tail(L, depth):
    rng = np.random.default_rng(L + depth)
    n = min(L // (3 * depth + 1), 400)  # pairs of lists that meet in one element
    for wrong in range(0, n, max(1, n // 24)):
        order = rng.permutation(L)
        succ = np.full(L, -2, dtype=np.int32)
        heads, at = [], 0
        for i in range(n):
            a, b = order[at:at + depth], order[at + depth:at + 2 * depth]
            tail = order[at + 2 * depth:at + 2 * depth + 1]
            at += 2 * depth + 1
            for part, meets in ((a, True), (b, i == wrong)):
                succ[part[:-1]] = part[1:]
                succ[part[-1]] = tail[0] if meets else -1
                heads.append(part[0])
            succ[tail] = -1
        assert _flagged(succ, np.array(heads, dtype=np.int32)), (L, depth, wrong)


@pytest.mark.parametrize("L,nlists", [(9000, 2000), (30000, 1500), (30000, 12000)])
def test_many_heads_name_a_list_twice(L, nlists):
    rng = np.random.default_rng(nlists)
    succ, heads, _ = _chain(rng.permutation(L), nlists, L)
    for at in range(0, nlists, nlists // 16):
        assert _flagged(succ, np.append(heads, heads[at])), (L, nlists, at)
