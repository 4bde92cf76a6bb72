"""Graphs whose union-find fits one workgroup's LDS: the sizes where the list is
no longer offered whole, the largest vertex count, answers that the one launch
cannot finish, and ids out of range wherever they stand.  Bridges, classes and
bridge trees must equal the oracle's."""
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


def dev(e):
    return torch.from_numpy(np.ascontiguousarray(e, dtype=np.int32).reshape(-1, 2)).cuda()


@pytest.fixture(scope="module", params=[1, 0], ids=["gpu_final_step", "host_search"])
def ctx(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07346_amd as br
    c = br.Context(0)
    c.set_final_step(request.param)
    c.set_profiling(1)
    yield c
    c.close()


def check(ctx, e, V, name, M=3, certificate=True):
    e = np.ascontiguousarray(e, dtype=np.int32).reshape(-1, 2)
    d = dev(e)
    want = oracle.bridges(e, V)
    say(name, "V=%d E=%d bridges %d" % (V, len(e), len(want)))
    assert np.array_equal(ctx.find(d, V, M), want), name
    assert ctx.profile()["plan_kind"] == 2
    wl, wt = oracle.bridge_tree(e, V)
    lab, t = ctx.bridge_tree(d, V, M)
    assert np.array_equal(lab, wl) and np.array_equal(t, wt), name
    lab, n = ctx.two_edge_components(d, V, M)
    assert np.array_equal(lab, wl) and n == np.unique(wl).shape[0], name
    if certificate:
        f1, f2 = ctx.cert_build(d, V, M)
        assert oracle.check_certificate(f1.cpu().numpy(), f2.cpu().numpy(), e, V) == [], name


def mixed(V, E, rng):
    """Random edges over most vertices, the others pendant or in small pieces."""
    core = max(1, V - V // 8)
    e = rng.integers(0, core, size=(E, 2))
    pend = min(V - core, E // 4)
    e[:pend, 0] = core + np.arange(pend)
    return e[rng.permutation(E)]


# one workgroup up to 8,192 vertices (rows of 3V edges up to 4,096, else 2V)
@pytest.mark.parametrize("V", [1, 2, 100, 2049, 4096, 4097, 8192, 8193, 40_943, 40_944])
def test_list_lengths(ctx, V):
    rng = np.random.default_rng(V)
    whole = max(16_384, min(8 * V, 32_768))               # offered whole up to here
    for E in (1, 511, 1025, whole - 1, whole, whole + 1, 2 * whole + 513, 9 * whole + 7):
        check(ctx, mixed(V, E, rng), V, "mixed")


def test_answers_left_to_the_other_step(ctx):
    rng = np.random.default_rng(1)
    for V in (4097, 4098, 4099, 6000):                    # rings: a core of V - 1 vertices
        p = rng.permutation(V)
        check(ctx, np.stack([p, np.roll(p, 1)], 1), V, "ring")
    for V in (16_385, 16_386, 16_387, 20_000):            # trees of V - 1 bridges
        i = np.arange(1, V)
        p = rng.permutation(V)
        e = np.stack([p[i], p[(rng.random(V - 1) * i).astype(np.int64)]], 1)
        check(ctx, e, V, "tree")
        check(ctx, np.concatenate([e, e[:3]]), V, "tree with copies")


def test_orders_and_lists(ctx):
    g = graphgen.planted(11, k=60, vc=30_000, p=0.15, n_extra=4, n_pend=500)
    order = np.lexsort((g.edges[:, 1], g.edges[:, 0]))
    check(ctx, g.edges[order], g.V, "sorted")
    d = dev(g.edges)
    for lo, hi in ((1, g.E), (3, g.E - 1), (5, 30_000)):
        assert np.array_equal(ctx.find(d[lo:hi], g.V), oracle.bridges(g.edges[lo:hi].copy(), g.V))
    want = oracle.bridges(g.edges, g.V)
    for cut in (1, 777, g.E // 2 + 1, g.E - 1):
        f1, f2 = ctx.cert_merge(d[:cut], d[cut:], g.V)
        s = torch.cat([f1, f2]).cpu().numpy()
        assert s.shape[0] <= 2 * (g.V - 1) and np.array_equal(oracle.bridges(s, g.V), want), cut
    s = graphgen.config("small")
    f1, f2 = ctx.cert_merge(dev(s.edges[:5000]), dev(s.edges[5000:]), s.V)
    assert np.array_equal(oracle.bridges(torch.cat([f1, f2]).cpu().numpy(), s.V), oracle.bridges(s.edges, s.V))


def test_ids_out_of_range_anywhere(ctx):
    import paper_2108_07346_amd as br
    rng = np.random.default_rng(4)
    for E in (20_000, 200_000):
        base = mixed(3000, E, rng).astype(np.int32)
        for at in [0, 511, 512, E - 1] + rng.integers(0, E, size=6).tolist():
            for bad in (3000, -1):
                e = base.copy()
                e[at, at % 2] = bad
                with pytest.raises(br.BridgeError) as ei:
                    ctx.find(dev(e), 3000)
                assert ei.value.code == br.BR_ERANGE, at
                with pytest.raises(br.BridgeError) as ei:
                    ctx.two_edge_components(dev(e), 3000)
                assert ei.value.code == br.BR_ERANGE, at
        check(ctx, base, 3000, "still usable")
