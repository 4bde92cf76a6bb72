"""The one-pass certificate (the whole list certified at once): the limits of
its stages and of the code widths of its table, lists in sorted order, unaligned
and concatenated lists, and ids out of range wherever they stand in the list.
Every bridge set must equal the oracle's."""
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


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07346_amd as br
    c = br.Context(0)
    c.set_profiling(1)
    yield c
    c.close()


def check(ctx, e, V, M=16, certificate=False):
    d = dev(e)
    want = oracle.bridges(np.ascontiguousarray(e, dtype=np.int32), V)
    assert np.array_equal(ctx.find(d, V, M), want), (V, len(e))
    assert ctx.profile()["plan_kind"] == 3
    if certificate:
        f1, f2 = ctx.cert_build(d, V, M)
        assert oracle.check_certificate(f1.cpu().numpy(), f2.cpu().numpy(), np.ascontiguousarray(e, dtype=np.int32), V) == []
    return d, want


# the stages change at 3 V, 4 V and 16 V edges
@pytest.mark.parametrize("E", [1, 511, 513, 3 * 45_001, 3 * 45_001 + 1, 4 * 45_001, 4 * 45_001 + 1, 16 * 45_001, 16 * 45_001 + 1, 20 * 45_001 + 77])
def test_stage_limits(ctx, monkeypatch, E):
    monkeypatch.setenv("BR_FUSE", "1")
    V = 45_001
    rng = np.random.default_rng(E)
    e = rng.integers(0, V - 2_000, size=(E, 2))
    pend = min(E // 2, 2_000)
    e[:pend, 0] = np.arange(V - pend, V)                  # pendant vertices among random edges
    check(ctx, e[rng.permutation(E)], V, certificate=True)


# largest V of each code width (16, 8, 4, 2, 1 bits, then no table), and one more
@pytest.mark.parametrize("V", [73_600, 73_601, 147_200, 147_201, 294_400, 294_401, 588_800, 588_801, 1_177_600, 1_177_601])
def test_table_limits(ctx, V):
    k = V // 256                                          # more clusters than the narrow codes can name
    g = graphgen.planted(V, k=k, vc=V - 300, p=0.15, n_extra=7, n_pend=300)
    assert g.V == V and g.E > 16 * V
    say("V=%d E=%d" % (V, g.E))
    check(ctx, g.edges, V)
    if V < 80_000:
        order = np.lexsort((g.edges[:, 1], g.edges[:, 0]))   # no row of the list stands for the whole
        check(ctx, g.edges[order], V, certificate=True)


def test_unaligned_and_concatenated_lists(ctx):
    g = graphgen.planted(5, k=200, vc=50_000, p=0.2, n_extra=3, n_pend=400)
    d = dev(g.edges)
    for lo, hi in ((1, g.E), (3, g.E - 1)):               # 8-byte aligned starts, odd ends
        assert np.array_equal(ctx.find(d[lo:hi], g.V, 3), oracle.bridges(g.edges[lo:hi].copy(), g.V))
    want = oracle.bridges(g.edges, g.V)
    for cut in (1, 777, g.E // 2 + 1, g.E - 1, g.E):
        f1, f2 = ctx.cert_merge(d[:cut], d[cut:], g.V)
        s = torch.cat([f1, f2]).cpu().numpy()
        assert s.shape[0] <= 2 * (g.V - 1) and np.array_equal(oracle.bridges(s, g.V), want), cut


def test_ids_out_of_range_anywhere(ctx):
    import paper_2108_07346_amd as br
    g = graphgen.planted(6, k=200, vc=50_000, p=0.2, n_extra=3, n_pend=400)
    rng = np.random.default_rng(6)
    for at in [0, 1, 511, 512, g.E - 1] + rng.integers(0, g.E, size=12).tolist():
        for bad in (g.V, -1):
            e = g.edges.copy()
            e[at, at % 2] = bad
            with pytest.raises(br.BridgeError) as ei:
                ctx.find(dev(e), g.V, 8)
            assert ei.value.code == br.BR_ERANGE, at
    check(ctx, g.edges, g.V)                              # still usable


def test_loops_and_parallel_edges(ctx):
    # every edge of a dense graph three times over, loops in between
    g = graphgen.planted(7, k=180, vc=45_000, p=0.1, n_extra=0, n_pend=500)
    loops = np.repeat(np.arange(0, g.V, 3), 2).reshape(-1, 2)
    rng = np.random.default_rng(7)
    e = np.concatenate([g.edges, g.edges[:, ::-1], g.edges, loops])
    check(ctx, e[rng.permutation(len(e))], g.V, certificate=True)
    e = np.concatenate([g.edges, loops])
    check(ctx, e[rng.permutation(len(e))], g.V)
