"""Ranking of long Euler tours through splitters: the limit at which it starts,
one tour of every arc, tours shorter than a splitter's group, trees that end
inside one, and depths from one to the whole list.  Against the oracle."""
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


def forest(kind, V, rng):
    i = np.arange(1, V)
    if kind == "path":
        e = np.stack([i - 1, i], 1)
    elif kind == "star":
        e = np.stack([np.zeros(V - 1, np.int64), i], 1)
    elif kind == "caterpillar":
        e = np.stack([np.where(i % 2 == 1, i - 1, i - 2), i], 1)
    elif kind == "random":
        e = np.stack([(rng.random(V - 1) * i).astype(np.int64), i], 1)
    else:                                              # trees of `kind` vertices
        e = np.stack([i - 1, i], 1)[i % kind != 0]
    return e


@pytest.mark.parametrize("V", [80_001, 80_002, 262_145, 262_146])
@pytest.mark.parametrize("kind", ["path", "star", "caterpillar", "random", 2, 3, 8, 9, 17, 1000])
def test_forests(ctx, V, kind):
    rng = np.random.default_rng(V)
    for order in ("as made", "relabelled and shuffled"):
        e = forest(kind, V, rng)
        if order != "as made":
            e = rng.permutation(V)[e][rng.permutation(len(e))]
        # some trees get edges that close cycles
        extra = e[rng.integers(0, len(e), size=50)]
        e = np.ascontiguousarray(np.concatenate([e, extra[:25], np.stack([extra[:25, 0], extra[25:, 0]], 1)]), np.int32)
        say(kind, V, order)
        d = torch.from_numpy(e).cuda()
        for _ in range(2):
            assert np.array_equal(ctx.find(d, V), oracle.bridges(e, V)), (kind, V, order)
        assert np.array_equal(ctx.articulation_points(d, V), oracle.articulation_points(e, V)), (kind, V, order)
