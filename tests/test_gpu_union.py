"""Batched graphs past the small kernel's 4,096 vertices: one query over their
disjoint union, beside the small ones.  Empty graphs, single graphs, limits of
the size classes, and an id that is valid in a neighbour but not in its own
graph.  Against the oracle."""
import sys

import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", params=[1, 0], ids=["gpu_final_step", "host_search"])
def ctx(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07346_amd as br
    c = br.Context(0)
    c.set_final_step(request.param)
    yield c
    c.close()


def pack(graphs):
    off = np.concatenate([[0], np.cumsum([len(e) for e, _ in graphs])]).astype(np.int64)
    e = np.concatenate([np.asarray(g, dtype=np.int32).reshape(-1, 2) for g, _ in graphs])
    return torch.from_numpy(np.ascontiguousarray(e)).cuda(), off, np.array([V for _, V in graphs], dtype=np.int32)


def check(ctx, graphs, name):
    d, off, V = pack(graphs)
    say(name, len(graphs), "graphs, E", int(off[-1]))
    pairs, boff = ctx.find_batched(d, off, V, 8192)
    for i, (e, v) in enumerate(graphs):
        want = oracle.bridges(np.ascontiguousarray(e, dtype=np.int32).reshape(-1, 2), int(v))
        assert np.array_equal(pairs[boff[i]:boff[i + 1]], want), (name, i, v)


def sizes(rng, Vs, f):
    out = []
    for V in Vs:
        k = max(1, V // 400)
        g = graphgen.planted(int(rng.integers(1 << 30)), k=k, vc=max(k, V - V // 20), p=min(1.0, f / max(1, V // k)),
                             n_extra=k // 30, n_pend=V - max(k, V - V // 20))
        out.append((g.edges, V))
    return out


def test_classes_and_limits(ctx):
    rng = np.random.default_rng(1)
    check(ctx, sizes(rng, [4095, 4096, 4097, 40_943, 40_944, 40_945, 100, 5000], 30), "limits")
    check(ctx, sizes(rng, [9000], 60), "one graph")
    check(ctx, sizes(rng, rng.integers(4097, 12_000, size=40), 20), "many")
    none = np.zeros((0, 2), np.int32)
    check(ctx, [(none, 5000), (none, 1), (none, 9000)], "no edges")
    check(ctx, sizes(rng, [6000], 40) + [(none, 7000), (np.array([[0, 6999]]), 7000)] + sizes(rng, [50, 8000], 40), "some empty")


def test_sparse_and_hard_unions(ctx):
    rng = np.random.default_rng(2)
    graphs = []
    for V in (5000, 20_000, 40_944):
        graphs.append((rng.integers(0, V, size=(int(1.4 * V), 2)), V))
        p = rng.permutation(V)
        graphs.append((np.stack([p, np.roll(p, 1)], 1), V))                # a ring: no bridges
        graphs.append((np.stack([p[:-1], p[1:]], 1), V))                   # a path: all bridges
    check(ctx, graphs, "random, rings, paths")


def test_ids_of_a_neighbour(ctx):
    import paper_2108_07346_amd as br
    rng = np.random.default_rng(3)
    graphs = sizes(rng, [5000, 6000, 7000], 30)
    for g in range(3):
        for bad in (graphs[g][1], -1):
            e = [x[0].copy() for x in graphs]
            e[g][len(e[g]) // 2, 1] = bad                                  # a vertex of the next graph in the union
            d, off, V = pack([(a, x[1]) for a, x in zip(e, graphs)])
            with pytest.raises(br.BridgeError) as ei:
                ctx.find_batched(d, off, V, 8192)
            assert ei.value.code == br.BR_ERANGE
    check(ctx, graphs, "still usable")
