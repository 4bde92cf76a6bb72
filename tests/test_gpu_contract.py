"""The final step over the contracted certificate: what crosses the components
of F' is a forest, has cycles with trees hanging from them, or is too large for
one workgroup (then the tour-based step answers).  Bridges, classes and bridge
trees must equal the oracle's."""
import itertools
import sys

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07346_amd as br
    c = br.Context(0)
    yield c
    c.close()


def blow_up(h, n, s, rng):
    """Every vertex of the graph h (n vertices) replaced by a complete graph of
    s vertices, ids relabelled, edges shuffled: (edges, V)."""
    inner = np.array(list(itertools.combinations(range(s), 2)), dtype=np.int64).reshape(-1, 2)
    e = (inner[None] + s * np.arange(n)[:, None, None]).reshape(-1, 2)
    h = np.asarray(h, dtype=np.int64).reshape(-1, 2)
    e = np.concatenate([e, h * s + rng.integers(0, s, size=h.shape)])
    e = rng.permutation(n * s)[e][rng.permutation(len(e))]
    return e.astype(np.int32), n * s


def tree(n, rng):
    i = np.arange(1, n)
    return np.stack([i, (rng.random(n - 1) * i).astype(np.int64)], 1)


def ring(n):
    return np.stack([np.arange(n), (np.arange(n) + 1) % n], 1)


def check(ctx, e, V, name, M=5):
    d = torch.from_numpy(np.ascontiguousarray(e)).cuda()
    want = oracle.bridges(e, V)
    say(name, "V=%d E=%d bridges %d" % (V, len(e), len(want)))
    assert np.array_equal(ctx.find(d, V, M), want), name
    wl, wt = oracle.bridge_tree(e, V)
    lab, n = ctx.two_edge_components(d, V, M)
    assert np.array_equal(lab, wl) and n == np.unique(wl).shape[0], name
    lab, t = ctx.bridge_tree(d, V, M)
    assert np.array_equal(lab, wl) and np.array_equal(t, wt), name


def shapes(n, rng):
    yield "tree", tree(n, rng)
    yield "ring", ring(n)
    k = max(2, n // 3)
    yield "ring with trees", np.concatenate([ring(k), np.stack([np.arange(k, n), (rng.random(n - k) * np.arange(k, n)).astype(np.int64)], 1)])
    yield "tree and chords", np.concatenate([tree(n, rng), rng.integers(0, n, size=(5, 2))])
    yield "long path with chords", np.concatenate([np.stack([np.arange(n - 1), np.arange(1, n)], 1),
                                                   [[n // 5, n // 3], [n // 2, n - 1]]])
    yield "star", np.stack([np.arange(1, n), np.zeros(n - 1, np.int64)], 1)
    yield "random", rng.integers(0, n, size=(n, 2))
    yield "pieces", np.concatenate([tree(n // 2, rng), ring(n - n // 2) + n // 2])


@pytest.mark.parametrize("n", [2, 3, 65, 1025])
def test_shapes(ctx, n):
    rng = np.random.default_rng(n)
    for name, h in shapes(n, rng):
        check(ctx, *blow_up(h, n, 14, rng), name)


# the core takes at most 4,096 vertices (a ring of n blocks loses one to F'),
# H at most 16,384 edges and vertices
@pytest.mark.parametrize("n", [4096, 4097, 4098, 4099])
def test_core_limit(ctx, n):
    rng = np.random.default_rng(n)
    check(ctx, *blow_up(ring(n), n, 14, rng), "ring")
    k = n - 2000                                          # trees hanging from the ring do not count
    h = np.concatenate([ring(n), np.stack([np.arange(n, n + k), rng.integers(0, n, size=k)], 1)])
    check(ctx, *blow_up(h, n + k, 14, rng), "ring with trees")


@pytest.mark.parametrize("n", [16383, 16384, 16385, 16386])
def test_size_limit(ctx, n):
    rng = np.random.default_rng(n)
    check(ctx, *blow_up(tree(n, rng), n, 14, rng), "tree")
    check(ctx, *blow_up(np.concatenate([tree(n, rng), [[0, n - 1]]]), n, 14, rng), "tree and a chord")


def test_small_graphs_of_any_density(ctx, monkeypatch):
    # up to 4,096 vertices the contracted step always runs first
    monkeypatch.setenv("BR_FUSE", "1")
    rng = np.random.default_rng(3)
    for t in range(60):
        V = int(rng.integers(1, 300)) if t < 50 else int(rng.integers(3000, 4097))
        e = rng.integers(0, V, size=(int(rng.integers(1, 4 * V)), 2)).astype(np.int32)
        check(ctx, e, V, "random t=%d" % t)
    for V in (2, 50, 4096):
        for name, h in shapes(V, rng):
            check(ctx, h.astype(np.int32), V, name)


# sparse lists at the edges per vertex from which the contraction is tried
@pytest.mark.parametrize("V, E", [(20_000, 60_000), (20_000, 59_999), (262_144, 786_432), (262_145, 786_435),
                                  (300_000, 1_200_000), (300_000, 1_199_999)])
def test_sparse_limits(ctx, V, E):
    rng = np.random.default_rng(E)
    check(ctx, rng.integers(0, V, size=(E, 2)).astype(np.int32), V, "random")
    # a tree takes a third of the edges: every edge of it is a bridge, more than the contraction holds at the larger sizes
    n = E // 3
    t = tree(min(n, V // 2), rng)
    e = np.concatenate([t, V // 2 + rng.integers(0, V - V // 2, size=(E - len(t), 2))])
    check(ctx, rng.permutation(V)[e][rng.permutation(E)].astype(np.int32), V, "tree and random")
