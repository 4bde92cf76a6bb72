"""Canonical order on the device: many keys, few keys, vertices with more keys
than a run holds, and the limits of each.  Against the oracle."""
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


def check(ctx, e, V, name):
    e = np.ascontiguousarray(e, dtype=np.int32)
    d = torch.from_numpy(e).cuda()
    want = oracle.bridges(e, V)
    say(name, "V=%d E=%d bridges %d" % (V, len(e), len(want)))
    assert np.array_equal(ctx.find(d, V), want), name
    wl, wt = oracle.bridge_tree(e, V)
    lab, t = ctx.bridge_tree(d, V)
    assert np.array_equal(lab, wl) and np.array_equal(t, wt), name


# one tree of `bridges` edges beside a long cycle: the device's order starts at 8,192 keys
@pytest.mark.parametrize("bridges", [1, 8191, 8192, 8193, 100_000])
def test_number_of_keys(ctx, bridges):
    rng = np.random.default_rng(bridges)
    V = 150_000
    i = np.arange(1, bridges + 1)
    tree = np.stack([i, (rng.random(bridges) * i).astype(np.int64)], 1)
    c = np.arange(bridges + 1, V)
    e = np.concatenate([tree, np.stack([c, np.roll(c, 1)], 1)])
    check(ctx, rng.permutation(V)[e][rng.permutation(len(e))], V, "tree and ring")


# hubs with as many bridges as a run holds, one more, and many; as the smaller
# and as the larger end
@pytest.mark.parametrize("leaves", [64, 65, 20_000])
@pytest.mark.parametrize("low", [True, False])
def test_hubs(ctx, leaves, low):
    rng = np.random.default_rng(leaves)
    V, hubs = 200_000, max(1, 20_000 // leaves)
    h = np.arange(hubs) if low else V - 1 - np.arange(hubs)
    rest = np.setdiff1d(np.arange(V), h)[rng.permutation(V - hubs)]
    star = np.stack([np.repeat(h, leaves), rest[:hubs * leaves]], 1)
    path = np.stack([h[:-1], h[1:]], 1)
    more = rest[hubs * leaves:]
    tail = np.stack([more[:-1], more[1:]], 1)
    e = np.concatenate([star, path, tail])
    check(ctx, e[rng.permutation(len(e))], V, "hubs")


@pytest.mark.parametrize("V", [(1 << 17) - 1, 1 << 17, 1_000_003])
def test_random_sparse(ctx, V):
    rng = np.random.default_rng(V)
    check(ctx, rng.integers(0, V, size=(int(1.5 * V), 2)), V, "random")
