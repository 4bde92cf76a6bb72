"""Articulation points of lists long enough for two rounds (rows of the list
through the block rules, then the edges of the rest that join different
groups): blocks that share cut vertices, sorted lists, codes of each width, more
remaining edges than their list holds, ids out of range.  Against the oracle."""
import itertools
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


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07346_amd as br
    c = br.Context(0)
    yield c
    c.close()


def check(ctx, e, V, name):
    e = np.ascontiguousarray(e, dtype=np.int32)
    want = oracle.articulation_points(e, V)
    say(name, "V=%d E=%d cut vertices %d" % (V, len(e), len(want)))
    got = ctx.articulation_points(torch.from_numpy(e).cuda(), V)
    assert np.array_equal(got, want), name


def chain(n, s, rng, relabel=True):
    """n complete graphs of s vertices, each sharing one vertex with an earlier one."""
    inner = np.array(list(itertools.combinations(range(s), 2)))
    ids = np.zeros((n, s), dtype=np.int64)
    ids[0] = np.arange(s)
    for i in range(1, n):
        ids[i, 1:] = s + (i - 1) * (s - 1) + np.arange(s - 1)
        ids[i, 0] = rng.integers(0, s + (i - 1) * (s - 1))
    V = s + (n - 1) * (s - 1)
    e = ids[:, inner].reshape(-1, 2)
    if relabel:
        e = rng.permutation(V)[e][rng.permutation(len(e))]
    return e, V


# 16-, 8- and 4-bit codes, more blocks than the narrow ones can name
@pytest.mark.parametrize("n,s", [(40, 180), (700, 60), (1500, 52), (2000, 80), (4000, 60)])
def test_chains_of_cliques(ctx, n, s):
    rng = np.random.default_rng(n)
    e, V = chain(n, s, rng)
    assert len(e) > 16 * V and len(e) >= 1 << 19
    check(ctx, e, V, "shuffled")
    e, V = chain(n, s, rng, relabel=False)
    check(ctx, e, V, "in order")


def test_planted(ctx):
    for seed, k, vc, p in ((1, 30, 9_000, 0.4), (2, 300, 76_000, 0.3)):
        g = graphgen.planted(seed, k=k, vc=vc, p=p, n_extra=6, n_pend=700)
        check(ctx, g.edges, g.V, "planted")
        check(ctx, g.edges[np.lexsort((g.edges[:, 1], g.edges[:, 0]))], g.V, "planted, sorted")


@pytest.mark.parametrize("hub", [0, 29_999])
def test_more_remaining_edges_than_the_list_holds(ctx, hub):
    # copies of a star's edges: those of the root never share a group
    rng = np.random.default_rng(5)
    V = 30_000
    leaf = np.setdiff1d(np.arange(V), [hub])
    star = np.stack([np.full(V - 1, hub), leaf], 1)
    some = np.stack([leaf[0:200:2], leaf[1:200:2]], 1)
    e = np.concatenate([np.repeat(star, 20, axis=0), some])
    check(ctx, e[rng.permutation(len(e))], V, "star")


def test_ids_out_of_range(ctx):
    import paper_2108_07346_amd as br
    rng = np.random.default_rng(6)
    e, V = chain(40, 180, rng)
    for at in [0, len(e) - 1] + rng.integers(0, len(e), size=6).tolist():
        bad = e.astype(np.int32)
        bad[at, 1] = V
        with pytest.raises(br.BridgeError) as ei:
            ctx.articulation_points(torch.from_numpy(bad).cuda(), V)
        assert ei.value.code == br.BR_ERANGE
    check(ctx, e, V, "still usable")
