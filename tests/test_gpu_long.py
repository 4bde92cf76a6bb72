"""Batched graphs with many edges per vertex: some rows of the list certified
first, the others on copies of their state.  Edge counts around the rule's
limits and the rows' and runs' ends, lists in which the first rows say nothing
about the others (so the runs keep the most they can), the two final steps, and
an id out of range in a row that only the second launch reads.  Against the
oracle."""
import sys

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
C = 1024


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


def blocks(rng, V, E, k):
    """E edges inside k blocks of the vertices, with a path of bridges between them"""
    cuts = np.sort(rng.choice(np.arange(1, V), size=min(k, V) - 1, replace=False)) if min(k, V) > 1 else np.zeros(0, np.int64)
    lo = np.concatenate([[0], cuts])
    hi = np.concatenate([cuts, [V]])
    b = rng.integers(0, len(lo), size=E)
    e = np.stack([rng.integers(lo[b], hi[b]), rng.integers(lo[b], hi[b])], 1)
    e[: len(lo) - 1] = np.stack([lo[:-1], lo[1:]], 1)[: E]
    return rng.permutation(V)[rng.permutation(e)].astype(np.int32)


def check(ctx, graphs, name):
    off = np.concatenate([[0], np.cumsum([len(e) for e, _ in graphs])]).astype(np.int64)
    d = torch.from_numpy(np.ascontiguousarray(np.concatenate([e for e, _ in graphs]))).cuda()
    say(name, len(graphs), "graphs, E", int(off[-1]))
    pairs, boff = ctx.find_batched(d, off, np.array([v for _, v in graphs], np.int32), C)
    for i, (e, v) in enumerate(graphs):
        want = oracle.bridges(np.ascontiguousarray(e), int(v))
        assert np.array_equal(pairs[boff[i]:boff[i + 1]], want), (name, i, v, len(e))


def test_around_the_rule(ctx):
    rng = np.random.default_rng(1)
    for V in (2, 3, 511, 513, 2048, 4095, 4096):
        least = max(2048, 8 * V)
        graphs = []
        for E in (least - 1, least, least + 1, least + 63, least + 65, 3 * least + 7, 32_767, 32_769, 65_536 + least):
            if E >= least - 1:
                graphs.append((blocks(rng, V, E, 5), V))
        check(ctx, graphs, f"V={V}")


def test_sorted_lists(ctx):
    rng = np.random.default_rng(2)
    graphs = []
    for V, E in ((4096, 200_000), (1000, 150_001), (4096, 65_536)):
        e = blocks(rng, V, E, 40)
        graphs.append((e[np.lexsort((e[:, 1], e[:, 0]))], V))
        # the rows taken first hold one repeated edge: every other edge survives
        r = np.arange(len(e)) // 64
        f = e.copy()
        f[r % (E // ((6 if E >= 128 * V else 4) * V)) == 0] = e[0]
        graphs.append((f, V))
    check(ctx, graphs, "sorted, repeated")


def test_out_of_range(ctx):
    import paper_2108_07346_amd as br
    rng = np.random.default_rng(3)
    V, E = 300, 20_000
    e = blocks(rng, V, E, 3)
    for at, bad in ((64 + 5, V), (E - 1, -1), (0, V)):
        f = e.copy()
        f[at, 1] = bad
        d = torch.from_numpy(f).cuda()
        with pytest.raises(br.BridgeError):
            ctx.find_batched(d, np.array([0, E]), np.array([V], np.int32), C)
    check(ctx, [(e, V)], "after an error")
