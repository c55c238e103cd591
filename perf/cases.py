"""The work the ranking library is timed on: one case per way it is called.

A case is a dict of plain values. `kind` names the entry point:
  rank    lr_rank over one input, `family` saying how its lists run through
          memory; rank output, with the root output where `root` is set
  psum    lr_prefix_sum with `weight` "i32" or "i64"; sums, and ranks and
          roots where `all` is set
  tree    lr_euler_tree: depth, preorder number and subtree size of every
          vertex of a random recursive tree from its Euler tour
  batch   lr_rank_batch over `count` independent lists of 2^lo .. 2^hi elements
  graph   the same requests replayed through a captured batch graph

Families (the instance families of the paper, as in workloads/): "random",
one list in random order; "forest", lists of mean length 64 plus four long
ones; "block", one list whose blocks of 4096 ids are walked one after another
in random order (most links local); "gamma", the identity order with a share
`gamma` of its positions permuted.

Inputs are drawn on the device from the seed alone. The program keeps its
workspace and its output arrays between calls, as a serving loop would.
"""
import math

import numpy as np
import torch

import paper_2606_09318_amd as lr

DEV = "cuda"
BLOCK = 4096


def listed():
    return [
        # a request of the smallest useful size: the call's fixed cost
        dict(name="rank_1k", kind="rank", family="random", n=1000, root=True),
        # a small ragged list, below every size the planner splits a level for
        dict(name="rank_20k", kind="rank", family="random", n=20011, root=True),
        # the ordinary single call: one random list of 2^20 elements
        dict(name="rank_1m", kind="rank", family="random", n=1 << 20, root=True),
        # many short lists and a few long ones, ragged size, both outputs
        dict(name="rank_forest_5m", kind="rank", family="forest", n=5000003, root=True),
        # a list stored mostly in list order (local links)
        dict(name="rank_block_67m", kind="rank", family="block", n=67108879, root=False),
        # the largest list of the benchmark, rank output alone
        dict(name="rank_268m", kind="rank", family="random", n=1 << 28, root=False),
        # small weighted list, int32 weights, sums alone
        dict(name="psum_i32_100k", kind="psum", family="random", n=100003, weight="i32", all=False),
        # the benchmark's weighted forest: int64 weights, every output
        dict(name="psum_i64_forest_134m", kind="psum", family="forest", n=1 << 27, weight="i64", all=True),
        # tree computations on a middling and on the benchmark's tree
        dict(name="tree_1m", kind="tree", V=1000003),
        dict(name="tree_67m", kind="tree", V=1 << 26),
        # a serving batch: 64 lists of 2^10 .. 2^22 elements in one call
        dict(name="batch_64", kind="batch", count=64, lo=10, hi=22, root=True),
        # a serving loop's small batches, replayed from a captured graph
        dict(name="graph_16", kind="graph", count=16, lo=10, hi=16, root=False),
    ]


def _size(rng, lo, hi):
    return int(2.0 ** rng.uniform(lo, hi)) | (rng.random() < 0.5)


def draw(rng):
    kind = rng.choice(["rank", "rank", "rank", "psum", "psum", "tree", "batch", "graph"])
    if kind == "tree":
        return dict(kind=kind, V=_size(rng, 10, 24))
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(2, 100), lo=10, hi=rng.choice([14, 18, 21]), root=rng.random() < 0.5)
    if kind == "graph":
        return dict(kind=kind, count=rng.randint(1, 32), lo=10, hi=rng.choice([13, 16, 18]), root=rng.random() < 0.5)
    family = rng.choice(["random", "random", "forest", "block", "gamma"])
    c = dict(kind=kind, family=family)
    if family == "gamma":
        c["gamma"] = round(rng.choice([0.003, 0.03, 0.1, 0.3]) * rng.uniform(0.7, 1.4), 5)
    if kind == "rank":
        c.update(n=_size(rng, 9, 26.5), root=rng.random() < 0.5)
    else:
        c.update(n=_size(rng, 9, 25.5), weight=rng.choice(["i32", "i64"]), all=rng.random() < 0.5)
    return c


# ------------------------------------------------------------------ inputs --

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _order(family, n, g, gamma=0.0):
    """The ids in visiting order (int64)."""
    if family == "block":
        nb = (n + BLOCK - 1) // BLOCK
        first = torch.randperm(nb, device=DEV, generator=g) * BLOCK
        within = torch.rand((nb, BLOCK), device=DEV, generator=g).argsort(dim=1)
        order = (first[:, None] + within).reshape(-1)
        return order[order < n]
    if family == "gamma":
        order = torch.arange(n, device=DEV)
        pos = torch.randperm(n, device=DEV, generator=g)[: int(round(gamma * n))]
        pos = pos.sort().values
        order[pos] = pos[torch.randperm(pos.numel(), device=DEV, generator=g)]
        return order
    return torch.randperm(n, device=DEV, generator=g)


def _ends(family, n, g):
    """Which positions of the order end a list (the last always does)."""
    if family == "forest":
        ends = torch.rand(n, device=DEV, generator=g) < 1.0 / 64.0
        for i in range(4):  # four long lists at the front, n / 64 elements each
            ends[i * (n // 64):(i + 1) * (n // 64)] = False
            if n // 64:
                ends[(i + 1) * (n // 64) - 1] = True
    else:
        ends = torch.zeros(n, dtype=torch.bool, device=DEV)
    ends[n - 1] = True
    return ends


def _lists(case, seed):
    """(order, ends, weights or None) of a rank or psum case."""
    g = _gen(seed)
    order = _order(case["family"], case["n"], g, case.get("gamma", 0.0))
    ends = _ends(case["family"], case["n"], g)
    w = None
    if case["kind"] == "psum":
        dt = torch.int32 if case["weight"] == "i32" else torch.int64
        w = torch.randint(-1000, 1001, (case["n"],), dtype=dt, device=DEV, generator=g)
    return order, ends, w


def _link(order, ends):
    succ = torch.empty(order.numel(), dtype=torch.int32, device=DEV)
    nxt = torch.where(ends, order, torch.roll(order, -1))
    succ[order] = nxt.to(torch.int32)
    return succ


def _request_sizes(case):
    r = np.random.default_rng(case["count"])
    return [int(2.0 ** u) for u in r.uniform(case["lo"], case["hi"], case["count"])]


def _request_order(i, n, seed):
    return _order("random" if i % 2 == 0 else "block", n, _gen(seed * 1000 + i))


def _tree(case, seed):
    """(parent, first child, next sibling) of a random recursive tree, children
    in ascending order; V marks none."""
    V = case["V"]
    g = _gen(seed)
    v = torch.arange(1, V, device=DEV)
    parent = torch.zeros(V, dtype=torch.int64, device=DEV)
    parent[1:] = torch.minimum((torch.rand(V - 1, device=DEV, generator=g, dtype=torch.float64) * v).long(), v - 1)
    kids = parent[1:].sort(stable=True)
    child = kids.indices + 1
    first = torch.full((V,), V, dtype=torch.int64, device=DEV)
    sibling = torch.full((V,), V, dtype=torch.int64, device=DEV)
    lead = torch.ones(V - 1, dtype=torch.bool, device=DEV)
    lead[1:] = kids.values[1:] != kids.values[:-1]
    first[kids.values[lead]] = child[lead]
    same = ~lead[1:]
    sibling[child[:-1][same]] = child[1:][same]
    return parent, first, sibling, g


def _tour(case, seed):
    """Successors of the tour's arcs and every vertex's down and up arc (arcs
    numbered in random order)."""
    V = case["V"]
    parent, first, sibling, g = _tree(case, seed)
    arc = torch.randperm(2 * (V - 1), device=DEV, generator=g)
    down = torch.zeros(V, dtype=torch.int64, device=DEV)
    up = torch.zeros(V, dtype=torch.int64, device=DEV)
    down[1:], up[1:] = arc[0::2], arc[1::2]
    succ = torch.empty(2 * (V - 1), dtype=torch.int32, device=DEV)
    has = first[1:] < V
    succ[down[1:]] = torch.where(has, down[first[1:].clamp(max=V - 1)], up[1:]).to(torch.int32)
    has = sibling[1:] < V
    back = torch.where(parent[1:] == 0, up[1:], up[parent[1:]])  # from the last child of the root: the tour ends
    succ[up[1:]] = torch.where(has, down[sibling[1:].clamp(max=V - 1)], back).to(torch.int32)
    return succ, down.to(torch.int32), up.to(torch.int32)


def _i32(n):
    return torch.empty(n, dtype=torch.int32, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("rank", "psum"):
        n = case["n"]
        order, ends, w = _lists(case, seed)
        st = dict(kind=kind, succ=_link(order, ends), weight=w)
        del order, ends
        if kind == "rank":
            st.update(rank=_i32(n), root=_i32(n) if case["root"] else None,
                      ws=lr.workspace(lr.lr_workspace_bytes(n)))
        else:
            wt = lr.LR_W_I32 if case["weight"] == "i32" else lr.LR_W_I64
            st.update(sum=torch.empty(n, dtype=torch.int64, device=DEV), rank=_i32(n) if case["all"] else None,
                      root=_i32(n) if case["all"] else None, ws=lr.workspace(lr.lr_workspace_bytes(n, wt)))
        return st
    if kind == "tree":
        V = case["V"]
        succ, down, up = _tour(case, seed)
        return dict(kind=kind, succ=succ, down=down, up=up, V=V, depth=_i32(V), preorder=_i32(V), size=_i32(V),
                    ws=lr.workspace(lr.lr_euler_tree_workspace_bytes(V)))
    # the requests' outputs are slices of one array each for ranks and roots
    sizes = _request_sizes(case)
    rank, root = _i32(sum(sizes)), _i32(sum(sizes)) if case["root"] else None
    items, at = [], 0
    for i, n in enumerate(sizes):
        order = _request_order(i, n, seed)
        ends = torch.zeros(n, dtype=torch.bool, device=DEV)
        ends[n - 1] = True
        items.append((_link(order, ends), rank[at:at + n], root[at:at + n] if case["root"] else None))
        at += n
    reqs = lr.requests(items)
    st = dict(kind=kind, items=items, reqs=reqs, count=len(items), rank=rank, root=root)
    if kind == "batch":
        st["ws"] = lr.workspace(lr.lr_batch_workspace_bytes(reqs, len(items)))
    else:
        cap = 1 << math.ceil(math.log2(case["count"] << case["hi"]))  # what the loop may be handed at once
        cfg = lr.batch_graph_config(cap, case["count"], case["root"])
        st["graph"] = lr.BatchGraph(cfg, lr.workspace(lr.lr_batch_graph_workspace_bytes(cfg)))
    return st


def run(state):
    kind = state["kind"]
    if kind == "rank":
        s = lr.lr_rank(state["succ"], state["rank"], state["root"], state["ws"])
    elif kind == "psum":
        s = lr.lr_prefix_sum(state["succ"], state["weight"], state["sum"], state["rank"], state["root"], state["ws"])
    elif kind == "tree":
        s = lr.lr_euler_tree(state["succ"], state["down"], state["up"], state["V"], 0, state["depth"],
                             state["preorder"], state["size"], state["ws"])
    elif kind == "batch":
        s = lr.lr_rank_batch(state["reqs"], state["count"], state["ws"])
    else:
        s = state["graph"].launch(state["reqs"], state["count"])
    if s:
        raise lr.LrError(s, kind)
    if kind == "psum":
        outs = (state["sum"], state["rank"], state["root"])
    elif kind == "tree":
        outs = (state["depth"], state["preorder"], state["size"])
    else:
        outs = (state["rank"], state["root"])
    return [t for t in outs if t is not None]


def work(case):
    """Bytes: every input array once, every output once. Operations: one
    addition per element and summed output."""
    kind = case["kind"]
    if kind == "tree":
        V = case["V"]
        return dict(bytes=4 * 2 * (V - 1) + 8 * V + 12 * V, flops=4 * V)
    if kind in ("batch", "graph"):
        n = sum(_request_sizes(case))
        return dict(bytes=(12 if case["root"] else 8) * n, flops=n)
    n = case["n"]
    if kind == "rank":
        return dict(bytes=(12 if case["root"] else 8) * n, flops=n)
    per = 4 + (4 if case["weight"] == "i32" else 8) + 8 + (8 if case["all"] else 0)
    return dict(bytes=per * n, flops=2 * n)


# ------------------------------------------------------------------- exact --

def _solve(order, ends, w=None):
    """(rank, root, sum) by position in the order."""
    n = order.numel()
    j = torch.arange(n, device=DEV)
    e = torch.where(ends, j, n).flip(0).cummin(0).values.flip(0)  # where the position's list ends
    rank = torch.empty(n, dtype=torch.int32, device=DEV)
    root = torch.empty(n, dtype=torch.int32, device=DEV)
    rank[order] = (e - j).to(torch.int32)
    root[order] = order[e].to(torch.int32)
    if w is None:
        return rank, root, None
    x = torch.where(ends, 0, w[order].to(torch.int64))
    c = x.cumsum(0)
    total = torch.empty(n, dtype=torch.int64, device=DEV)
    total[order] = c[e] - c + x
    return rank, root, total


def exact(case, seed):
    kind = case["kind"]
    if kind in ("rank", "psum"):
        order, ends, w = _lists(case, seed)
        rank, root, total = _solve(order, ends, w)
        if kind == "rank":
            return [rank, root] if case["root"] else [rank]
        return [total, rank, root] if case["all"] else [total]
    if kind == "tree":
        V = case["V"]
        parent, _, _, _ = _tree(case, seed)
        depth = torch.zeros(V, dtype=torch.int64, device=DEV)
        while True:  # a random recursive tree is a few dozen levels deep
            d = depth[parent] + 1
            d[0] = 0
            if torch.equal(d, depth):
                break
            depth = d
        by_depth = depth.sort(stable=True)
        cuts = torch.searchsorted(by_depth.values, torch.arange(int(depth.max()) + 2, device=DEV)).tolist()
        level = [by_depth.indices[cuts[i]:cuts[i + 1]] for i in range(len(cuts) - 1)]
        size = torch.ones(V, dtype=torch.int64, device=DEV)
        for vs in reversed(level[1:]):
            size.index_add_(0, parent[vs], size[vs])
        # position among the siblings: the sizes of the earlier ones
        kids = parent[1:].sort(stable=True)
        child = kids.indices + 1
        before = size[child].cumsum(0) - size[child]
        lead = torch.ones(V - 1, dtype=torch.bool, device=DEV)
        lead[1:] = kids.values[1:] != kids.values[:-1]
        start = torch.where(lead, before, 0).cummax(0).values
        offset = torch.zeros(V, dtype=torch.int64, device=DEV)
        offset[child] = before - start
        pre = torch.zeros(V, dtype=torch.int64, device=DEV)
        for vs in level[1:]:
            pre[vs] = pre[parent[vs]] + 1 + offset[vs]
        return [t.to(torch.int32) for t in (depth, pre, size)]
    ranks, roots = [], []
    for i, n in enumerate(_request_sizes(case)):
        order = _request_order(i, n, seed)
        ends = torch.zeros(n, dtype=torch.bool, device=DEV)
        ends[n - 1] = True
        rank, root, _ = _solve(order, ends)
        ranks.append(rank)
        roots.append(root)
    return [torch.cat(ranks), torch.cat(roots)] if case["root"] else [torch.cat(ranks)]
