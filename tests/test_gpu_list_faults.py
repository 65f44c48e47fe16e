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
