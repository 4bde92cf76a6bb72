"""Which branch answers on either side of a rule's limit.  Every branch gives the
same answer and most have another to fall back on, so answers alone do not tell
whether a limit lies where it is meant to, or whether a branch is reached."""
import ctypes

import numpy as np
import pytest

import oracle
from test_gpu_contract import blow_up, ring, tree
from test_gpu_orders import path, relabelled

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

HOST, TOURS, CONTRACTED, AGAIN, IN_LAUNCH = range(5)


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07346_amd as br
    c = br.Context(0)
    yield c
    c.close()


def route(ctx):
    out = (ctypes.c_int64 * 5)()
    assert ctx._lib.br_route(ctx._h, out) == 0
    return dict(zip(("final", "past", "longs", "in_unions", "alone"), out))


def final(ctx, e, V, M=5):
    """The final step that answered bridges, classes and the tree (the same one)."""
    d = torch.from_numpy(np.ascontiguousarray(e, dtype=np.int32)).cuda()
    assert np.array_equal(ctx.find(d, V, M), oracle.bridges(e, V))
    r = route(ctx)["final"]
    wl, wt = oracle.bridge_tree(e, V)
    assert np.array_equal(ctx.two_edge_components(d, V, M)[0], wl)
    assert route(ctx)["final"] == r
    lab, t = ctx.bridge_tree(d, V, M)
    assert np.array_equal(lab, wl) and np.array_equal(t, wt)
    assert route(ctx)["final"] == r
    print("V=%d E=%d final step %d" % (V, len(e), r), flush=True)
    return r


@pytest.mark.parametrize("n,want", [(4096, CONTRACTED), (4097, CONTRACTED), (4098, TOURS)])
def test_core_limit(ctx, n, want):
    # a ring of n blocks loses one to F': its core has n - 1 vertices, 4,096 at most
    assert final(ctx, *blow_up(ring(n), n, 14, np.random.default_rng(n))) == want


@pytest.mark.parametrize("n,want", [(16_383, CONTRACTED), (16_384, CONTRACTED), (16_385, TOURS)])
def test_size_limit(ctx, n, want):
    rng = np.random.default_rng(n)
    assert final(ctx, *blow_up(tree(n, rng), n, 14, rng)) == want
    # the chord closes a ring, which loses one edge to F' and with it a vertex
    h = np.concatenate([tree(n + 1, rng), [[0, n]]])
    assert final(ctx, *blow_up(h, n + 1, 14, rng)) == want


@pytest.mark.parametrize("V,E,want", [(20_000, 60_000, CONTRACTED), (20_000, 59_999, TOURS), (262_144, 786_432, CONTRACTED),
                                      (262_145, 786_435, TOURS), (300_000, 1_200_000, CONTRACTED), (300_000, 1_199_999, TOURS)])
def test_sparse_limits(ctx, V, E, want):
    assert final(ctx, np.random.default_rng(E).integers(0, V, size=(E, 2)), V) == want


@pytest.mark.parametrize("E,want", [(16_384, IN_LAUNCH), (16_385, CONTRACTED)])
def test_whole_lists(ctx, E, want):
    # E <= 16,384, or up to 8V edges where that is more
    assert final(ctx, np.random.default_rng(E).integers(0, 1000, size=(E, 2)), 1000) == want


def test_long_chains(ctx):
    # every edge six times: shuffled ids leave chains of a few steps, ids in order some
    # of more than 64
    V = 50_000
    e = np.repeat(path(V), 6, 0)
    assert final(ctx, e, V) == AGAIN
    assert final(ctx, relabelled(e, V), V) == CONTRACTED


@pytest.mark.parametrize("V,E,past", [(40_000, 640_000, 0), (40_000, 640_001, 1), (20_000, 524_287, 0), (20_000, 524_288, 1),
                                      (1000, 16_384, 0), (1000, 16_385, 1)])
def test_tables(ctx, V, E, past):
    # past 8,192 vertices: more than 16V edges, and 2^19; up to there: lists not offered whole
    e = np.random.default_rng(E).integers(0, V, size=(E, 2)).astype(np.int32)
    assert np.array_equal(ctx.find(torch.from_numpy(e).cuda(), V, 3), oracle.bridges(e, V))
    assert route(ctx)["past"] == past


@pytest.mark.parametrize("V,C,E,is_long", [(500, 1000, 3999, 0), (500, 1000, 4000, 1), (100, 1000, 2047, 0), (100, 1000, 2048, 1),
                                           (100, 3000, 3000, 0), (100, 3000, 3001, 1)])
def test_long_graphs_of_a_batch(ctx, V, C, E, is_long):
    # more than a chunk, and at least 8V and 2,048 edges
    e = [np.random.default_rng(E + i).integers(0, V, size=(E, 2)).astype(np.int32) for i in range(3)]
    d = torch.from_numpy(np.concatenate(e)).cuda()
    pairs, off = ctx.find_batched(d, np.arange(4, dtype=np.int64) * E, np.full(3, V, np.int32), C)
    assert all(np.array_equal(pairs[off[i]:off[i + 1]], oracle.bridges(e[i], V)) for i in range(3))
    assert route(ctx)["longs"] == 3 * is_long


@pytest.mark.parametrize("Vs,per,want", [((5000,), 20, (0, 1, 1)), ((5000, 6000), 20, (2, 0, 2)), ((5000, 6000), 10, (2, 0, 0)),
                                         ((100, 4096), 20, (0, 0, None)), ((100, 4097, 4096, 40_944), 17, (2, 0, 2))])
def test_unions_of_a_batch(ctx, Vs, per, want):
    # (in unions, alone, the list's long part: past a table per graph from 16V edges)
    e = [np.random.default_rng(V).integers(0, V, size=(per * V, 2)).astype(np.int32) for V in Vs]
    off = np.concatenate([[0], np.cumsum([len(x) for x in e])]).astype(np.int64)
    pairs, boff = ctx.find_batched(torch.from_numpy(np.concatenate(e)).cuda(), off, np.array(Vs, np.int32), 1 << 20)
    for i, V in enumerate(Vs):
        assert np.array_equal(pairs[boff[i]:boff[i + 1]], oracle.bridges(e[i], V)), V
    r = route(ctx)
    assert (r["in_unions"], r["alone"]) == want[:2]
    if want[2] is not None and want[0]:
        assert r["past"] == want[2]
