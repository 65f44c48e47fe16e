"""Performance cases of the Euler-tour library, as a program that uses it
calls it: trees built and queried, resident trees, edge lists, plain and
weighted lists, bridges of one graph, and batches of trees and graphs.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same
ranges, ``prepare`` makes a case's inputs on the GPU from a seed, ``run`` is
one pass, ``work`` the bytes a pass cannot do without, and ``exact`` the same
results computed with torch alone (pointer doubling in 64-bit integers).

Inputs follow the repository's generators: grasp trees (node i picks its
parent among the g nodes before it) under a random relabelling, uniform
queries, sparse graphs of blobs joined by planted chains, seeded random
permutations cut into lists, batches of log-uniform sizes.
"""
import math

import numpy as np
import torch

import paper_2103_15217_amd as et

DEV = "cuda"


def listed():
    return [
        # one small instance at a time, e.g. a served job: latency and launches
        {"name": "tree_small", "kind": "tree", "n": 1000, "grasp": 0, "q": 1024, "stats": False},
        # a deep tree of ordinary size with its depth / preorder / size tables taken out
        {"name": "tree_deep", "kind": "tree", "n": 1000003, "grasp": 1000, "q": 262144, "stats": True},
        # the benchmark's size: a shallow random tree, one query per node
        {"name": "tree_large", "kind": "tree", "n": 1 << 24, "grasp": 0, "q": 1 << 24, "stats": False},
        # a tree kept resident that only answers queries
        {"name": "queries", "kind": "queries", "n": 1 << 22, "grasp": 64, "q": 5000001},
        # a tree given as unordered edges (the DCEL construction), rooted and tabulated
        {"name": "tree_edges", "kind": "edges", "n": 3000001, "grasp": 0, "q": 65536, "stats": True},
        # list ranking on its own, at the benchmark's length
        {"name": "list_large", "kind": "list", "n": 1 << 25, "heads": 1, "weighted": False, "rank": True},
        # weighted ranking of many lists at once, with unused slots
        {"name": "list_scan", "kind": "list", "n": 1000003, "heads": 1000, "weighted": True, "rank": True},
        # bridges of one small sparse graph, the count read back: latency and launches
        {"name": "graph_small", "kind": "graph", "n": 5000, "m": 20000, "chains": 16, "max_chain": 8,
         "count": True},
        # bridges at the benchmark's size
        {"name": "graph_large", "kind": "graph", "n": 1 << 22, "m": 1 << 25, "chains": 4096, "max_chain": 512,
         "count": False},
        # many trees of uneven size in one batched build and query
        {"name": "forest", "kind": "forest", "trees": 1000, "log2_min": 6.0, "log2_max": 18.0, "log2_qmin": 10.0,
         "log2_qmax": 14.0},
        # many small trees built and queried in one launch
        {"name": "small_trees", "kind": "small_trees", "trees": 1000, "log2_min": 6.0, "log2_max": 12.0,
         "log2_qmin": 10.0, "log2_qmax": 14.0},
        # many small graphs in one call (one launch when every graph fits, else the batched kernels)
        {"name": "graphs", "kind": "graphs", "graphs": 1300, "log2_min": 3.0, "log2_max": 10.0, "degree": 4},
    ]


def _log(rng, lo, hi):
    """An integer log-uniform on [lo, hi]."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["tree", "tree", "queries", "edges", "list", "list", "graph", "graph", "forest", "small_trees",
                       "graphs", "graphs"])
    if kind == "tree":
        n = _log(rng, 200, 12_000_000)
        return {"kind": kind, "n": n, "grasp": rng.choice([0, 0, 1, 64, 1000]), "q": _log(rng, 200, max(n, 4096)),
                "stats": rng.random() < 0.5}
    if kind == "queries":
        return {"kind": kind, "n": _log(rng, 1000, 8_000_000), "grasp": rng.choice([0, 1, 64, 1000]),
                "q": _log(rng, 1000, 16_000_000)}
    if kind == "edges":
        n = _log(rng, 1000, 6_000_000)
        return {"kind": kind, "n": n, "grasp": rng.choice([0, 64, 1000]), "q": _log(rng, 1000, n), "stats": True}
    if kind == "list":
        n = _log(rng, 1000, 32_000_000)
        weighted = rng.random() < 0.5
        return {"kind": kind, "n": n, "heads": _log(rng, 1, max(1, n // 500)), "weighted": weighted,
                "rank": not weighted or rng.random() < 0.5}
    if kind == "graph":
        n = _log(rng, 500, 4_000_000)
        chains = _log(rng, 4, max(4, n // 1024))
        return {"kind": kind, "n": n, "m": int(n * rng.uniform(2.0, 8.0)), "chains": chains,
                "max_chain": max(2, min(512, n // (4 * chains))), "count": rng.random() < 0.5}
    if kind == "forest":
        return {"kind": kind, "trees": _log(rng, 16, 800), "log2_min": 6.0, "log2_max": rng.uniform(13.0, 17.5),
                "log2_qmin": 10.0, "log2_qmax": rng.uniform(11.0, 14.0)}
    if kind == "small_trees":
        return {"kind": kind, "trees": _log(rng, 3, 4000), "log2_min": rng.uniform(4.0, 6.0),
                "log2_max": rng.uniform(9.0, 12.0), "log2_qmin": 10.0, "log2_qmax": rng.uniform(11.0, 14.0)}
    return {"kind": "graphs", "graphs": _log(rng, 16, 4000), "log2_min": 3.0, "log2_max": rng.uniform(8.0, 12.0),
            "degree": rng.choice([3, 4, 8])}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _rand_below(hi, g):
    """A uniform integer in [0, hi[i]) per entry (0 where hi is 0)."""
    r = torch.rand(hi.shape, dtype=torch.float64, device=DEV, generator=g)
    return torch.minimum((r * hi).to(torch.int64), (hi - 1).clamp(min=0))


def _sizes(count, lo, hi, seed):
    """``count`` sizes spread evenly over the logarithm of [2^lo, 2^hi], in an order made from the seed."""
    s = np.floor(2.0 ** (lo + (hi - lo) * (np.arange(count) + 0.5) / count)).astype(np.int64)
    return np.random.default_rng([int(seed), count]).permutation(s)


def _offsets(sizes):
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)


def _relabel(base, size, total, g):
    """A random permutation of the ids inside every part: part k holds the ids [base[k], base[k] + size[k])."""
    if len(size) == 1:
        return torch.randperm(total, device=DEV, generator=g)
    part = torch.repeat_interleave(torch.arange(len(size), device=DEV), size)
    order = torch.argsort(part + torch.rand(total, dtype=torch.float64, device=DEV, generator=g))
    lab = torch.empty(total, dtype=torch.int64, device=DEV)
    lab[order] = torch.arange(total, device=DEV)
    return lab


def _grasp_forest(sizes, grasps, g):
    """Parents (global ids, -1 at the roots) of trees laid out back to back, before relabelling, and the tree of each id."""
    size = torch.as_tensor(sizes, device=DEV)
    grasp = torch.as_tensor([x if x else int(s) for x, s in zip(grasps, sizes)], device=DEV)
    base = torch.cumsum(size, 0) - size
    total = int(sizes.sum())
    part = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), size)
    local = torch.arange(total, device=DEV) - base[part]
    lo = (local - grasp[part]).clamp(min=0)
    par = base[part] + lo + _rand_below(local - lo, g)
    par[local == 0] = -1
    return par, part, base, size


def _trees(sizes, grasps, g):
    """Relabelled parents with local ids, -1 at the roots (int32), and the same with global ids."""
    par, part, base, size = _grasp_forest(sizes, grasps, g)
    lab = _relabel(base, size, par.numel(), g)
    glob = torch.empty_like(par)
    glob[lab] = torch.where(par < 0, par, lab[par.clamp(min=0)])
    local = torch.where(glob < 0, glob, glob - base[part])
    return local.to(torch.int32), glob


def _queries(sizes, counts, g):
    """Uniform local pairs, grouped by tree, and their tree ids."""
    tree = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), torch.as_tensor(counts, device=DEV))
    hi = torch.as_tensor(sizes, device=DEV)[tree]
    return _rand_below(hi, g).to(torch.int32), _rand_below(hi, g).to(torch.int32), tree.to(torch.int32)


def _csr(n, u, w):
    key = torch.sort(torch.cat([u * n + w, w * n + u]))[0]
    src = key // n
    row = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    row[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    return row.to(torch.int32), (key - src * n).to(torch.int32)


def _blob_edges(starts, sizes, extra, g):
    """Every blob's random recursive tree (parents, -1 at its first vertex) and ``extra[k]`` further pairs inside blob
    k, drawn uniformly (a few repeat an edge)."""
    nv = int(sizes.sum())
    sizes, starts = torch.as_tensor(sizes, device=DEV), torch.as_tensor(starts, device=DEV)
    blob = torch.repeat_interleave(torch.arange(sizes.numel(), device=DEV), sizes)
    local = torch.arange(nv, device=DEV) - starts[blob]
    par = starts[blob] + _rand_below(local, g)
    par[local == 0] = -1
    blob = torch.repeat_interleave(torch.arange(sizes.numel(), device=DEV), torch.as_tensor(extra, device=DEV))
    size = sizes[blob]
    u = _rand_below(size, g)
    w = (u + 1 + _rand_below(size - 1, g)) % size
    return par, starts[blob] + u, starts[blob] + w


def _graph(case, seed):
    """A sparse graph: blobs joined by planted chains (every eighth chain hangs loose, so the graph has several
    components), its CSR and the parents of one spanning forest."""
    g = _gen(seed)
    n, chains = case["n"], case["chains"]
    length = 1 + np.arange(chains, dtype=np.int64) * (case["max_chain"] - 1) // max(chains - 1, 1)
    length = np.random.default_rng([int(seed), 1]).permutation(length)
    nv = n - int((length - 1).sum())
    bounds = np.arange(chains + 2, dtype=np.int64) * nv // (chains + 1)
    starts, sizes = bounds[:-1], np.diff(bounds)
    extra = max(0, case["m"] - int(length.sum()) - (nv - chains - 1))
    par, u, w = _blob_edges(starts, sizes, np.diff(bounds * extra // nv), g)
    # chain k hangs the first vertex of blob k + 1 below a vertex of an earlier blob
    k = torch.arange(chains, device=DEV)
    top = _rand_below(torch.as_tensor(starts[1:], device=DEV), g)
    top = torch.where(k % 8 == 7, -1, top)
    par = torch.cat([par, torch.zeros(n - nv, dtype=torch.int64, device=DEV)])
    length = torch.as_tensor(length, device=DEV)
    first = nv + torch.cumsum(length - 1, 0) - (length - 1)
    inner = torch.arange(nv, n, device=DEV)
    owner = torch.repeat_interleave(k, length - 1)
    par[inner] = torch.where(inner == first[owner], top[owner], inner - 1)
    par[torch.as_tensor(starts[1:], device=DEV)] = torch.where(length > 1, first + length - 2, top)
    perm = torch.randperm(n, device=DEV, generator=g)
    forest = torch.empty_like(par)
    forest[perm] = torch.where(par < 0, par, perm[par.clamp(min=0)])
    child = torch.nonzero(forest >= 0)[:, 0]
    row, col = _csr(n, torch.cat([perm[u], child]), torch.cat([perm[w], forest[child]]))
    return row, col, forest


def _graphs(case, seed):
    """Connected sparse graphs back to back: the union's CSR, the forest's parents and the offsets."""
    g = _gen(seed)
    sizes = _sizes(case["graphs"], case["log2_min"], case["log2_max"], seed)
    voff = _offsets(sizes)
    n = int(voff[-1])
    par, u, w = _blob_edges(voff[:-1], sizes, sizes * (case["degree"] - 2) // 2, g)
    lab = _relabel(torch.as_tensor(voff[:-1], device=DEV), torch.as_tensor(sizes, device=DEV), n, g)
    forest = torch.empty_like(par)
    forest[lab] = torch.where(par < 0, par, lab[par.clamp(min=0)])
    child = torch.nonzero(forest >= 0)[:, 0]
    row, col = _csr(n, torch.cat([lab[u], child]), torch.cat([lab[w], forest[child]]))
    return row, col, forest, sizes, voff


def _list(case, seed):
    """A random permutation cut into lists, one slot in 64 unused: successors, heads, the order and each one's start in it."""
    g = _gen(seed)
    n, heads = case["n"], case["heads"]
    used = n - n // 64
    order = torch.randperm(n, device=DEV, generator=g)[:used]
    start = torch.arange(heads, device=DEV) * used // heads
    succ = torch.full((n,), -2, dtype=torch.int32, device=DEV)
    nxt = torch.roll(order, -1)
    nxt[(start - 1) % used] = -1
    succ[order] = nxt.to(torch.int32)
    weight = torch.randint(-(1 << 20), 1 << 20, (n,), device=DEV, generator=g, dtype=torch.int64).to(torch.int32)
    return succ, order[start].to(torch.int32), weight, order, start


_GRASPS = (1, 64, 0)


def _batch(case, seed):
    g = _gen(seed)
    sizes = _sizes(case["trees"], case["log2_min"], case["log2_max"], seed)
    counts = _sizes(case["trees"], case["log2_qmin"], case["log2_qmax"], seed + 1)
    parent, glob = _trees(sizes, [_GRASPS[i % 3] for i in range(len(sizes))], g)
    qx, qy, qt = _queries(sizes, counts, g)
    return sizes, counts, parent, glob, qx, qy, qt


def _edge_tree(case, seed):
    g = _gen(seed)
    parent, glob = _trees(np.array([case["n"]]), [case["grasp"]], g)
    qx, qy, _ = _queries([case["n"]], [case["q"]], g)
    return parent, glob, qx, qy, g


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    if kind in ("tree", "queries", "edges"):
        parent, glob, s["qx"], s["qy"], g = _edge_tree(case, seed)
        s["stats"] = case.get("stats", False)
        if kind == "tree":
            s["parent"] = parent
        elif kind == "queries":
            s["tree"] = et.et_tree_build(parent)
        else:
            child = torch.nonzero(glob >= 0)[:, 0]
            child = child[torch.randperm(child.numel(), device=DEV, generator=g)]
            flip = torch.rand(child.numel(), device=DEV, generator=g) < 0.5
            s["u"] = torch.where(flip, child, glob[child]).to(torch.int32)
            s["v"] = torch.where(flip, glob[child], child).to(torch.int32)
            s["n"], s["root"] = case["n"], int(torch.argmin(glob))
    elif kind == "list":
        s["succ"], s["heads"], s["weight"], _, _ = _list(case, seed)
        s["weighted"], s["rank"] = case["weighted"], case["rank"]
    elif kind == "graph":
        s["row"], s["col"], _ = _graph(case, seed)
        s["count"] = case["count"]
    elif kind == "graphs":
        row, col, _, sizes, voff = _graphs(case, seed)
        soff = row[torch.as_tensor(voff, device=DEV)].to(torch.int64)
        # every graph's own row pointers, from 0
        at = torch.cat([torch.as_tensor(voff[:-1], device=DEV)[:, None], torch.as_tensor(voff[1:], device=DEV)[:, None]], 1)
        part = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), at[:, 1] - at[:, 0] + 1)
        rows = row[torch.arange(part.numel(), device=DEV) - part].to(torch.int64) - soff[part]
        base = torch.repeat_interleave(at[:, 0], torch.diff(soff))
        slots = torch.diff(soff).cpu().numpy()
        s["args"] = {"row_ptr": rows.to(torch.int32), "col": (col - base).to(torch.int32),
                     "voff": torch.as_tensor(voff, device=DEV), "soff": soff, "slots": slots.tolist()}
        s["fits"] = int(sizes.max()) <= et.FUSED_MAX_VERTICES and int(slots.max()) <= et.FUSED_MAX_SLOTS
        if s["fits"]:
            s["args"]["vertices"] = sizes.tolist()
            s["args"]["order"] = torch.as_tensor(et.fused_graph_order(slots, sizes), device=DEV)
    else:
        sizes, counts, s["parent"], _, s["qx"], s["qy"], s["qt"] = _batch(case, seed)
        off, qoff = _offsets(sizes), _offsets(counts)
        s["off"], s["qoff"] = torch.as_tensor(off, device=DEV), torch.as_tensor(qoff, device=DEV)
        s["most"] = int(sizes.max())
        s["order"] = torch.as_tensor(et.fused_order(off, qoff), device=DEV) if s["most"] > 1024 else None
    return s


# ------------------------------------------------------------------ one pass

_STATS = ("depth", "pre", "size")


def run(s):
    kind = s["kind"]
    if kind == "queries":
        return s["tree"].lca(s["qx"], s["qy"])
    if kind in ("tree", "edges"):
        tree = et.et_tree_build(s["parent"]) if kind == "tree" else et.et_tree_build_edges(s["u"], s["v"], s["n"],
                                                                                          s["root"])
        out = {"lca": tree.lca(s["qx"], s["qy"])}
        if s["stats"]:
            out.update(tree.export(_STATS))
        tree.free()
        return out
    if kind == "list":
        if not s["weighted"]:
            return et.et_list_rank(s["succ"], s["heads"])
        return et.et_list_scan(s["succ"], s["weight"], s["heads"], rank=s["rank"])
    if kind == "graph":
        mask, count = et.et_bridges(s["row"], s["col"], count=s["count"])
        return (mask, count) if s["count"] else mask
    if kind == "graphs":
        mask, _, counts = (et.et_bridges_batch_fused if s["fits"] else et.et_bridges_batch)(**s["args"])
        return mask, counts
    if kind == "forest":
        tree = et.et_tree_build_batch(s["parent"], s["off"])
        out = tree.lca_batch(s["qt"], s["qx"], s["qy"])
        tree.free()
        return out
    return et.et_lca_batch_fused(s["parent"], s["off"], s["qoff"], s["qx"], s["qy"], s["most"], order=s["order"])


def work(case):
    """Each input read once and each output written once. There are no floating-point operations."""
    kind = case["kind"]
    if kind == "queries":  # the two nodes' table entries (inlabel, ascendant, depth) per query at most once per node
        nbytes = 12 * case["q"] + 12 * min(case["n"], 2 * case["q"])
    elif kind == "tree":
        nbytes = 4 * case["n"] + 12 * case["q"] + (12 * case["n"] if case["stats"] else 0)
    elif kind == "edges":
        nbytes = 8 * (case["n"] - 1) + 12 * case["q"] + (12 * case["n"] if case["stats"] else 0)
    elif kind == "list":
        n = case["n"]
        nbytes = 4 * n + 4 * case["heads"] + (8 * n if case["weighted"] else 0) + (4 * n if case["rank"] else 0)
    elif kind == "graph":
        nbytes = 4 * (case["n"] + 1) + 8 * case["m"] + case["m"] // 4
    elif kind == "graphs":
        n = int(_sizes(case["graphs"], case["log2_min"], case["log2_max"], 0).sum())
        nbytes = 4 * (n + case["graphs"]) + 4 * n * case["degree"] + n * case["degree"] // 8
    else:
        n = int(_sizes(case["trees"], case["log2_min"], case["log2_max"], 0).sum())
        q = int(_sizes(case["trees"], case["log2_qmin"], case["log2_qmax"], 0).sum())
        nbytes = 4 * n + (16 if kind == "forest" else 12) * q
    return {"bytes": nbytes, "flops": 0}


# ------------------------------------------------------------------ plain results

def _lift(parent):
    """Ancestors at distance 2^k for every k below log2 of the depth (the roots' own ids stay), int32."""
    ids = torch.arange(parent.numel(), device=DEV)
    anc = [torch.where(parent < 0, ids, parent).to(torch.int32)]
    while True:
        up = anc[-1][anc[-1].long()]
        if torch.equal(up, anc[-1]):
            return anc
        anc.append(up)


def _sum_up(value, parent, anc):
    """Per node the sum of ``value`` over its ancestors and itself (the roots' values are 0)."""
    acc = value.clone()
    for a in anc:
        acc = acc + acc[a.long()]
    return acc


def _sum_subtree(value, parent):
    """Per node the (wrapping) sum of ``value`` over its subtree."""
    n = parent.numel()
    acc = torch.cat([value, value.new_zeros(1)])  # an extra node above the roots takes what leaves the forest
    up = torch.cat([torch.where(parent < 0, n, parent), parent.new_full((1,), n)])
    while bool((up[:n] < n).any()):
        acc = acc.index_add(0, up, acc)
        acc[n] = 0
        up = up[up]
    return acc[:n]


def _depth(parent, anc):
    return _sum_up((parent >= 0).long(), parent, anc)


def _lca(parent, anc, depth, x, y):
    x, y = x.long(), y.long()
    swap = depth[x] < depth[y]
    x, y = torch.where(swap, y, x), torch.where(swap, x, y)
    diff = depth[x] - depth[y]
    for k in reversed(range(len(anc))):
        x = torch.where((diff >> k) & 1 == 1, anc[k][x].long(), x)
    for k in reversed(range(len(anc))):
        ax, ay = anc[k][x].long(), anc[k][y].long()
        x, y = torch.where(ax != ay, ax, x), torch.where(ax != ay, ay, y)
    return torch.where(x == y, x, anc[0][x].long())


def _stats(parent, anc, cyclic):
    """Depth, preorder and subtree size; children in ascending id order, or in cyclic order after the parent's id."""
    n = parent.numel()
    depth, size = _depth(parent, anc), _sum_subtree(torch.ones_like(parent), parent)
    ids = torch.arange(n, device=DEV)
    rank = ids
    if cyclic:  # a child's turn at its parent p: after p's own parent, around; ascending at the root
        grand = torch.where(parent < 0, -1, parent[parent.clamp(min=0)])
        rank = torch.where(grand < 0, ids, (ids - grand - 1) % n)
    order = torch.argsort(parent * n + rank)
    sz = size[order]
    before = torch.cumsum(sz, 0) - sz
    new = torch.ones(n, dtype=torch.bool, device=DEV)
    new[1:] = parent[order][1:] != parent[order][:-1]
    first = torch.cummax(torch.where(new, torch.arange(n, device=DEV), 0), 0)[0]
    step = torch.empty_like(parent)
    step[order] = 1 + before - before[first]
    return {"depth": depth, "pre": _sum_up(torch.where(parent < 0, 0, step), parent, anc), "size": size}


def _bridge_slots(row, col, forest, seed):
    """Which CSR slots are bridges: a forest edge is one iff no other edge leaves the child's subtree. Every other
    edge (a repeated copy is one) adds a random number at one end and takes it off at the other, so that the edges inside a subtree cancel."""
    n, nnz = forest.numel(), col.numel()
    src = torch.repeat_interleave(torch.arange(n, device=DEV), torch.diff(row.long()))
    dst = col.long()
    same = torch.zeros(nnz + 1, dtype=torch.bool, device=DEV)  # slot k repeats slot k - 1 (rows are sorted)
    same[1:-1] = (src[1:] == src[:-1]) & (dst[1:] == dst[:-1])
    tree = ((forest[src] == dst) | (forest[dst] == src)) & ~same[:-1]
    g = _gen(seed + 5)
    lo, hi = torch.minimum(src, dst), torch.maximum(src, dst)
    one = (src < dst) & ~tree
    r = torch.randint(1, 1 << 62, (nnz,), device=DEV, generator=g, dtype=torch.int64) * one
    value = torch.zeros(n, dtype=torch.int64, device=DEV).index_add(0, lo, r).index_add(0, hi, -r)
    alone = (_sum_subtree(value, forest) == 0) & (forest >= 0)
    child = torch.where(forest[src] == dst, src, dst)
    return tree & alone[child]


def _words(bit, on, count):
    """int32 words with the given bits set."""
    w = torch.zeros(count, dtype=torch.int64, device=DEV)
    w.index_add_(0, bit >> 5, on.long() << (bit & 31))
    return torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32)


def exact(case, seed):
    kind = case["kind"]
    i32 = torch.int32
    if kind in ("tree", "queries", "edges"):
        _, glob, qx, qy, _ = _edge_tree(case, seed)
        anc = _lift(glob)
        lca = _lca(glob, anc, _depth(glob, anc), qx, qy).to(i32)
        if kind == "queries":
            return lca
        out = {"lca": lca}
        if case["stats"]:
            out.update({k: v.to(i32) for k, v in _stats(glob, anc, kind == "edges").items()})
        return out
    if kind == "list":
        _, _, weight, order, start = _list(case, seed)
        at = torch.arange(order.numel(), device=DEV)
        head = start[torch.searchsorted(start, at, right=True) - 1]
        rank = torch.full((case["n"],), -1, dtype=i32, device=DEV)
        rank[order] = (at - head).to(i32)
        if not case["weighted"]:
            return rank
        w = weight[order].long()
        run_sum = torch.cumsum(w, 0)
        total = torch.zeros(case["n"], dtype=torch.int64, device=DEV)
        total[order] = run_sum - run_sum[head] + w[head]
        total = (((total + (1 << 31)) % (1 << 32)) - (1 << 31)).to(i32)
        return (total, rank) if case["rank"] else total
    if kind == "graph":
        row, col, forest = _graph(case, seed)
        bit = _bridge_slots(row, col, forest, seed)
        mask = _words(torch.arange(col.numel(), device=DEV), bit, max((col.numel() + 31) // 32, 1))
        return (mask, int(bit.sum()) // 2) if case["count"] else mask
    if kind == "graphs":
        row, col, forest, _, voff = _graphs(case, seed)
        bit = _bridge_slots(row, col, forest, seed)
        soff = row[torch.as_tensor(voff, device=DEV)].to(torch.int64)
        slots = torch.diff(soff)
        words = (slots + 31) // 32
        part = torch.repeat_interleave(torch.arange(slots.numel(), device=DEV), slots)
        at = 32 * (torch.cumsum(words, 0) - words)[part] + torch.arange(col.numel(), device=DEV) - soff[part]
        counts = torch.zeros(slots.numel(), dtype=torch.int64, device=DEV).index_add(0, part, bit.long()) // 2
        return _words(at, bit, int(words.sum())), counts
    sizes, _, _, glob, qx, qy, qt = _batch(case, seed)
    base = torch.as_tensor(_offsets(sizes)[:-1], device=DEV)[qt.long()]
    anc = _lift(glob)
    return (_lca(glob, anc, _depth(glob, anc), base + qx, base + qy) - base).to(i32)
