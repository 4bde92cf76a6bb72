"""The calls whose speed this library answers for, one pass of each.

Every case is a call (or a short run of calls) that a program using the
binding makes on graphs it has on the GPU.  The graphs are made on the GPU:
planted clusters joined by a tree with a few extra edges and pendant vertices
(the shape of the small, dense, large, batched and served workloads), or
uniform sparse multigraphs.  A case fixes the graph's structure; the seed
relabels its ids, shuffles its edges and picks their orientations, so the
inputs and outputs of two seeds differ while the counts (bridges, classes, cut
vertices) stay the same.

kinds
  find      bridges of one graph over M chunks (Context.find)
  tree      2-edge-connected classes and the bridge tree (Context.bridge_tree)
  classes   2-edge-connected classes alone (Context.two_edge_components)
  cut       articulation points (Context.articulation_points)
  batched   bridges of many packed graphs in one call (Context.find_batched)
  served    a burst of requests through a Server, all collected
  shards    certificates of the shards of an edge list, merged pairwise, and
            the bridges of the merged certificate (cert_build, cert_merge, find)
"""
import math

import numpy as np
import torch

import paper_2108_07346_amd as br


def _planted(name, kind, k, s, p, pend, extra, M, cross=0):
    return {"name": name, "kind": kind, "graph": "planted", "k": k, "s": s, "p": p, "pend": pend, "extra": extra,
            "cross": cross, "M": M}


def _sparse(name, kind, V, E, M):
    return {"name": name, "kind": kind, "graph": "sparse", "V": V, "E": E, "M": M}


def listed():
    return [
        # one small query, where launches and copies are all there is: the small
        # configuration (20 clusters of 100, M = 4)
        _planted("find_small", "find", 20, 100, 0.1, 30, 1, 4),
        # a mid-sized graph whose union-find still fits a CU's LDS, odd sizes,
        # as a serving program sends them
        _planted("find_mid", "find", 13, 947, 0.27, 34, 1, 15),
        # the dense configuration at the chunk count it is benchmarked at
        _planted("find_dense", "find", 256, 256, 0.5, 1000, 5, 16),
        # a sparse network (three edges per two vertices): most of the edges
        # are in the certificate and many of them are bridges
        _sparse("find_sparse", "find", 1_000_003, 1_500_007, 8),
        # the large configuration, the largest call: 1.03e9 edges, M = 4096
        _planted("find_large", "find", 1024, 256, 1.0, 5000, 0, 4096, 262_144 * 7_600 // 2),
        # classes and the bridge tree of the dense configuration
        _planted("tree_dense", "tree", 256, 256, 0.5, 1000, 5, 16),
        # classes of a sparse multigraph, one chunk: the whole path is
        # O(V) work with a label per vertex as output
        _sparse("classes_sparse", "classes", 400_009, 1_000_003, 1),
        # failure points of the dense configuration
        _planted("cut_dense", "cut", 256, 256, 0.5, 1000, 5, 1),
        # the batched configuration: 4,096 graphs of 64..4,096 vertices
        {"name": "batched_many", "kind": "batched", "G": 4096, "vlo": 64, "vhi": 4096, "plo": 0.05, "phi": 0.5},
        # fewer graphs of mixed size classes, some past the small kernel's 4,096
        {"name": "batched_mixed", "kind": "batched", "G": 150, "vlo": 100, "vhi": 24_000, "plo": 0.02, "phi": 0.1},
        # the served configuration: a burst of queries, V 256..131,072,
        # degree 64..2,048, all resident on the device
        {"name": "served_burst", "kind": "served", "n": 48, "vlo": 256, "vhi": 131_072, "dlo": 64, "dhi": 2048},
        # a list that arrives in shards: 10^7 edges over 10^5 vertices (the
        # figures' size) in 4 shards of 10 chunks
        dict(_planted("shards", "shards", 390, 256, 0.785, 160, 8, 10), shards=4),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.choice(["find", "find", "find", "find", "tree", "classes", "cut", "batched", "served", "shards"])
    if kind == "batched":
        vhi = _logint(rng, 300, 30_000)
        # about 2e8 edges at most
        g = min(4096, max(3, int(2e8 / (0.02 * vhi * vhi))))
        return {"kind": kind, "G": _logint(rng, 2, g), "vlo": rng.randint(20, 100), "vhi": vhi,
                "plo": 0.02, "phi": 0.1 if vhi > 4096 else 0.5}
    if kind == "served":
        return {"kind": kind, "n": _logint(rng, 4, 64), "vlo": 256, "vhi": _logint(rng, 1000, 131_072), "dlo": 16,
                "dhi": _logint(rng, 32, 1024)}
    if kind in ("find", "tree", "classes") and rng.random() < 0.4:
        V = _logint(rng, 200, 3_000_000)
        return {"kind": kind, "graph": "sparse", "V": V, "E": int(V * rng.uniform(0.6, 3.0)),
                "M": _logint(rng, 1, 64)}
    s = _logint(rng, 5, 700)
    V = _logint(rng, 100, 300_000)
    k = max(1, V // s)
    p = min(1.0, max(rng.uniform(0.05, 1.0), 6.0 / s))
    cap = 3e8 if kind == "find" else 3e7
    inner = k * s * (s - 1) / 2 * p
    if inner > cap:
        p = p * cap / inner
    cross = 0
    if kind == "find" and rng.random() < 0.5 and k > 1:
        cross = _logint(rng, 1, max(2, int(min(cap, 1500.0 * V))))
    c = _planted("", kind, k, s, p, rng.randint(3, max(3, V // 50)), rng.randint(0, max(1, k // 20)),
                 _logint(rng, 1, 4096) if kind == "find" else _logint(rng, 1, 64), cross)
    del c["name"]
    if kind == "shards":
        c["shards"] = rng.randint(2, 6)
    return c


# ---- inputs -----------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & ((1 << 62) - 1))
    return g


def _randint(g, hi, shape):
    return torch.randint(0, hi, shape, generator=g, device="cuda", dtype=torch.int32)


def _finish(e, V, g):
    """Relabel the ids, flip orientations, shuffle the list."""
    relabel = torch.randperm(V, generator=g, device="cuda").to(torch.int32)
    order = torch.randperm(e.shape[0], generator=g, device="cuda")
    e = e[order]
    del order
    out = torch.empty_like(e)
    for lo in range(0, e.shape[0], 1 << 27):       # in pieces: the index is 64-bit
        hi = min(lo + (1 << 27), e.shape[0])
        a = relabel[e[lo:hi].reshape(-1).long()].reshape(-1, 2)
        flip = torch.rand((hi - lo, 1), generator=g, device="cuda") < 0.5
        out[lo:hi] = torch.where(flip, a.flip(1), a)
    return out.contiguous()


def _planted_edges(g, k, s, p, pend, extra, cross):
    """k clusters of s vertices with inner edge probability p, a random tree of
    single edges between them, `extra` more such edges, `cross` uniform
    inter-cluster edges, `pend` pendant vertices: (V, edges before relabelling)."""
    parts = []
    if s > 1:
        iu = torch.triu_indices(s, s, 1, device="cuda", dtype=torch.int32)
        pairs = iu.shape[1]
        step = max(1, (1 << 27) // pairs)
        for lo in range(0, k, step):
            kb = min(step, k - lo)
            if p >= 1.0:
                c = torch.arange(lo, lo + kb, device="cuda", dtype=torch.int32).repeat_interleave(pairs)
                i = torch.arange(pairs, device="cuda").repeat(kb)
            else:
                hit = (torch.rand((kb, pairs), generator=g, device="cuda") < p).nonzero()
                c, i = hit[:, 0].to(torch.int32) + lo, hit[:, 1]
            parts.append(torch.stack([iu[0][i] + c * s, iu[1][i] + c * s], 1))
    if k > 1:
        # tree: cluster i > 0 to a random earlier one; extra: any two clusters
        i = torch.arange(1, k, device="cuda", dtype=torch.int32)
        j = (torch.rand(k - 1, generator=g, device="cuda") * i).to(torch.int32).clamp_(max=k - 2)
        j = torch.minimum(j, i - 1)
        parts.append(torch.stack([i * s + _randint(g, s, (k - 1,)), j * s + _randint(g, s, (k - 1,))], 1))
        for n in (extra, cross):
            for lo in range(0, n, 1 << 28):
                m = min(1 << 28, n - lo)
                a = _randint(g, k, (m,))
                b = (a + 1 + _randint(g, k - 1, (m,))) % k
                parts.append(torch.stack([a * s + _randint(g, s, (m,)), b * s + _randint(g, s, (m,))], 1))
    if pend:
        leaf = torch.arange(k * s, k * s + pend, device="cuda", dtype=torch.int32)
        parts.append(torch.stack([leaf, _randint(g, k * s, (pend,))], 1))
    if not parts:
        parts.append(torch.zeros((0, 2), device="cuda", dtype=torch.int32))
    return k * s + pend, torch.cat(parts)


def _structure():
    """The generator of the structure, the same for every seed."""
    return _gen(20_108)


def _graph(case, g):
    t = _structure()
    if case["graph"] == "sparse":
        V, e = case["V"], _randint(t, case["V"], (case["E"], 2))
    else:
        V, e = _planted_edges(t, case["k"], case["s"], case["p"], case["pend"], case["extra"], case["cross"])
    return V, _finish(e, V, g)


def _batch_sizes(case):
    """Vertex counts, clusters and probabilities of a batch: the same for every seed."""
    r = np.random.default_rng(case["G"] * 1_000_003 + case["vhi"])
    out = []
    for _ in range(case["G"]):
        V = max(2, int(round(math.exp(r.uniform(math.log(case["vlo"]), math.log(case["vhi"]))))))
        k = min(int(r.integers(2, 17)), max(1, V // 2))
        if V > 4096:
            k = max(k, V // 600)
        out.append((V, k, float(r.uniform(case["plo"], case["phi"])), int(r.uniform(0, 0.03) * (k - 1) + r.random())))
    return out


def _request_sizes(case):
    """(V, k, s, p) of the requests of a burst: the same for every seed."""
    r = np.random.default_rng(case["n"] * 7_919 + case["vhi"])
    out = []
    for _ in range(case["n"]):
        V = int(round(math.exp(r.uniform(math.log(case["vlo"]), math.log(case["vhi"])))))
        d = math.exp(r.uniform(math.log(case["dlo"]), math.log(case["dhi"])))
        s = min(V, max(256, int(2 * d)))
        out.append((V, max(1, V // s), s, min(1.0, d / (s - 1))))
    return out


def _many(case, g):
    """The graphs of a batch or a burst: [(V, edges)]."""
    out, t = [], _structure()
    if case["kind"] == "batched":
        for V, k, p, extra in _batch_sizes(case):
            s = V // k
            out.append(_planted_edges(t, k, s, p, V - k * s, extra, 0))
    else:
        for V, k, s, p in _request_sizes(case):
            out.append(_planted_edges(t, k, s, p, V - k * s + int(0.015 * V), int(0.02 * k), 0))
    return [(V, _finish(e, V, g)) for V, e in out]


# ---- the cases --------------------------------------------------------------

def prepare(case, seed):
    """What a program has before the call: the graphs on the GPU, its context."""
    g = _gen(seed)
    kind = case["kind"]
    st = {"case": case}
    if kind == "batched":
        graphs = _many(case, g)
        st["V"] = np.array([V for V, _ in graphs], dtype=np.int32)
        st["off"] = np.concatenate([[0], np.cumsum([e.shape[0] for _, e in graphs])]).astype(np.int64)
        st["edges"] = torch.cat([e for _, e in graphs]).contiguous()
        st["ctx"] = br.Context(0)
    elif kind == "served":
        st["graphs"] = _many(case, g)
        st["server"] = br.Server(0)
    else:
        V, e = _graph(case, g)
        st["V"] = V
        if kind == "shards":
            n, E = case["shards"], e.shape[0]
            st["shards"] = [e[i * E // n:(i + 1) * E // n].clone() for i in range(n)]
        else:
            st["edges"] = e
        st["ctx"] = br.Context(0)
    torch.cuda.synchronize()
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "find":
        return state["ctx"].find(state["edges"], state["V"], case["M"])
    if kind == "tree":
        return state["ctx"].bridge_tree(state["edges"], state["V"], case["M"])
    if kind == "classes":
        return state["ctx"].two_edge_components(state["edges"], state["V"], case["M"])
    if kind == "cut":
        return state["ctx"].articulation_points(state["edges"], state["V"])
    if kind == "batched":
        return state["ctx"].find_batched(state["edges"], state["off"], state["V"])
    if kind == "served":
        srv = state["server"]
        tickets = [srv.submit(e, V) for V, e in state["graphs"]]
        return [srv.wait(t, V) for t, (V, _) in zip(tickets, state["graphs"])]
    ctx, V = state["ctx"], state["V"]
    certs = [torch.cat(ctx.cert_build(e, V, case["M"])) for e in state["shards"]]
    while len(certs) > 1:
        nxt = [torch.cat(ctx.cert_merge(certs[i], certs[i + 1], V)) for i in range(0, len(certs) - 1, 2)]
        certs = nxt + certs[len(certs) - len(certs) % 2:]
    return ctx.find(certs[0], V)


def _sizes(case):
    """[(V, expected E)] of the graphs of a case."""
    def planted(k, s, p, pend, extra, cross):
        return k * s + pend, k * s * (s - 1) / 2 * min(p, 1.0) + max(0, k - 1) + pend + (extra + cross if k > 1 else 0)
    if case["kind"] == "batched":
        return [planted(k, V // k, p, V - k * (V // k), extra, 0) for V, k, p, extra in _batch_sizes(case)]
    if case["kind"] == "served":
        return [planted(k, s, p, V - k * s + int(0.015 * V), int(0.02 * k), 0) for V, k, s, p in _request_sizes(case)]
    if case["graph"] == "sparse":
        return [(case["V"], float(case["E"]))]
    return [planted(case["k"], case["s"], case["p"], case["pend"], case["extra"], case["cross"])]


def work(case):
    """Every edge read once (8 bytes); labels written where the call returns
    them; an integer operation per edge endpoint (no floating point)."""
    b = ops = 0.0
    for V, E in _sizes(case):
        b += 8 * E + (4 * V if case["kind"] in ("tree", "classes") else 0)
        ops += 2 * E
    return {"bytes": int(b), "flops": int(ops)}


# ---- what the outputs are, without the library ------------------------------

def _lowlink(V, e):
    """Depth-first search with low-links: (bridges as an edge mask, cut-vertex flags)."""
    n = e.shape[0]
    src = np.concatenate([e[:, 0], e[:, 1]])
    order = np.argsort(src, kind="stable")
    dst = np.concatenate([e[:, 1], e[:, 0]])[order].tolist()
    eid = (order % max(n, 1)).tolist()
    ptr = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=V))]).tolist()
    it = ptr[:V]
    disc, low = [-1] * V, [0] * V
    bridge, cut = np.zeros(n, bool), np.zeros(V, bool)
    clock = 0
    for r in range(V):
        if disc[r] >= 0:
            continue
        disc[r] = low[r] = clock
        clock += 1
        kids = 0
        stack = [(r, -1)]
        while stack:
            x, pe = stack[-1]
            if it[x] < ptr[x + 1]:
                a = it[x]
                it[x] = a + 1
                y, i = dst[a], eid[a]
                if i == pe or y == x:
                    continue
                if disc[y] < 0:
                    disc[y] = low[y] = clock
                    clock += 1
                    stack.append((y, i))
                elif disc[y] < low[x]:
                    low[x] = disc[y]
            else:
                stack.pop()
                if stack:
                    w = stack[-1][0]
                    if low[x] < low[w]:
                        low[w] = low[x]
                    if low[x] > disc[w]:
                        bridge[pe] = True
                    if w == r:
                        kids += 1
                    elif low[x] >= disc[w]:
                        cut[w] = True
        cut[r] = kids > 1
    return bridge, cut


def _sorted_pairs(e):
    e = np.sort(e, 1)
    return e[np.lexsort((e[:, 1], e[:, 0]))].astype(np.int32).reshape(-1, 2)


def _labels(V, e):
    """Smallest vertex of each vertex's component."""
    lab = np.arange(V)
    while True:
        m = np.minimum(lab[e[:, 0]], lab[e[:, 1]])
        new = lab.copy()
        for c in (0, 1):
            np.minimum.at(new, lab[e[:, c]], m)
            np.minimum.at(new, e[:, c], m)
        while True:
            nn = new[new]
            if np.array_equal(nn, new):
                break
            new = nn
        if np.array_equal(new, lab):
            return lab.astype(np.int32)
        lab = new


def exact(case, seed):
    """The outputs from a plain depth-first search; None where it would take long."""
    if sum(E + V for V, E in _sizes(case)) > 5e6:
        return None
    g = _gen(seed)
    if case["kind"] in ("batched", "served"):
        res = []
        for V, e in _many(case, g):
            e = e.cpu().numpy().astype(np.int64)
            res.append(_sorted_pairs(e[_lowlink(V, e)[0]]))
        if case["kind"] == "served":
            return res
        return np.concatenate(res), np.concatenate([[0], np.cumsum([len(r) for r in res])]).astype(np.int64)
    V, e = _graph(case, g)
    e = e.cpu().numpy().astype(np.int64)
    bridge, cut = _lowlink(V, e)
    if case["kind"] in ("find", "shards"):
        return _sorted_pairs(e[bridge])
    if case["kind"] == "cut":
        return np.flatnonzero(cut).astype(np.int32)
    lab = _labels(V, e[~bridge])
    if case["kind"] == "classes":
        return lab, int(np.unique(lab).shape[0])
    return lab, _sorted_pairs(lab[e[bridge]].astype(np.int64))
