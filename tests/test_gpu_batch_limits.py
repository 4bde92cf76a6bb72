"""Batches at the limits of memory and of the chunk count: what a batch of larger
graphs holds on the device beside its edge list, and which chunk sizes it takes."""
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
def br():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07346_amd as br
    return br


def dense_with_pendants(g, V, E, k):
    """E random edges over V - k vertices, then k pendant ones: the last k edges are
    the bridges (every other vertex has more than 2,000 edges)."""
    core = torch.randint(0, V - k, (E, 2), device="cuda", dtype=torch.int32)
    leaf = torch.arange(V - k, V, device="cuda", dtype=torch.int32)
    hook = torch.arange(k, device="cuda", dtype=torch.int32) * 7 + g
    return torch.cat([core, torch.stack([leaf, hook], 1)]), torch.stack([hook, leaf], 1).cpu().numpy()


@pytest.mark.parametrize("graphs,E,held", [
    (1, 30_000_000, 64),           # queried where it lies
    (12, 24_000_000, 1024 + 64),   # 2.3 GB of edges: unions of up to 1 GiB
    (3, 140_000_000, 64),          # each past that alone
])
def test_device_memory_of_larger_graphs(br, graphs, E, held):
    """MiB the context may hold after the call: the union's copy at most, and 64 for
    a query's workspace over 60,000 vertices (137 words for each are 33)."""
    torch.manual_seed(graphs)
    V, k = 5000, 9
    made = [dense_with_pendants(g, V, E, k) for g in range(graphs)]
    d = torch.cat([e for e, _ in made])
    want = [w for _, w in made]
    off = np.arange(graphs + 1, dtype=np.int64) * (E + k)
    del made
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    ctx = br.Context(0)
    warm = torch.zeros((1, 2), dtype=torch.int32, device="cuda")
    ctx.find_batched(warm, np.array([0, 1], np.int64), np.array([4], np.int32), 1 << 20)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    pairs, boff = ctx.find_batched(d, off, np.full(graphs, V, np.int32), 1 << 20)
    used = (free - torch.cuda.mem_get_info()[0]) / 2**20
    say("%d graphs of %d edges: %.0f MiB held" % (graphs, E, used))
    for g in range(graphs):
        assert np.array_equal(pairs[boff[g]:boff[g + 1]], want[g])
    ctx.close()
    assert used <= held


def test_unions_next_to_each_other(br):
    """Graphs on either side of the end of a union, an empty one and one of loops
    among them; ids out of range are still found."""
    rng = np.random.default_rng(3)
    V = [4097, 5000, 40_000, 4500, 9000, 4200, 100, 6000, 7000]
    E = [30_000_000, 60_000_000, 44_000_000, 0, 30_000, 4, 500, 2_000_000, 40_000]
    lists = [torch.randint(0, v - 3, (e, 2), device="cuda", dtype=torch.int32) for v, e in zip(V, E)]
    for v, e in zip(V, lists):
        if e.shape[0] > 10:
            e[5] = torch.tensor([v - 2, v - 1])
    lists[5][:] = 7
    off = np.concatenate([[0], np.cumsum(E)]).astype(np.int64)
    d = torch.cat(lists)
    ctx = br.Context(0)
    pairs, boff = ctx.find_batched(d, off, np.array(V, np.int32), 1 << 20)
    for g, (v, e) in enumerate(zip(V, E)):
        got = pairs[boff[g]:boff[g + 1]]
        if e == 0 or g == 5:
            assert len(got) == 0
        elif e <= 2_000_000:
            assert np.array_equal(got, oracle.bridges(lists[g].cpu().numpy(), v)), g
        else:
            assert np.array_equal(got, ctx.find(lists[g], v, 1)), g
    for g in (0, 2, 7):
        bad = d.clone()
        bad[int(off[g + 1]) - 1, 1] = V[g]
        with pytest.raises(br.BridgeError) as x:
            ctx.find_batched(bad, off, np.array(V, np.int32), 1 << 20)
        assert x.value.code == br.BR_ERANGE
    ctx.close()


@pytest.mark.parametrize("V", [100, 4096, 4097, 40_000])
def test_chunks_per_graph(br, V):
    """A graph of 2^20 chunks or more is refused, whether it would be split into them
    or not; one fewer is taken."""
    n = 1 << 20
    e = np.random.default_rng(V).integers(0, V, size=(n, 2)).astype(np.int32)
    d = torch.from_numpy(e).cuda()
    ctx = br.Context(0)
    Vs = np.array([V, 5], np.int32)
    with pytest.raises(br.BridgeError) as x:
        ctx.find_batched(d, np.array([0, n, n], np.int64), Vs, 1)
    assert x.value.code == br.BR_EINVAL
    for m, chunk in ((n, 2), (n - 1, 1)):
        pairs, off = ctx.find_batched(d[:m], np.array([0, m, m], np.int64), Vs, chunk)
        assert np.array_equal(pairs, oracle.bridges(e[:m], V)) and list(off) == [0, len(pairs), len(pairs)]
    ctx.close()
