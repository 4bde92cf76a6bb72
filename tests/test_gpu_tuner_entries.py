"""What the entries of the tuner's cache file select: each stored here by hand under
the key that the library gives for the graph's shape."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import json, sys
sys.path.insert(0, %r)
import numpy as np, torch, oracle
import paper_2108_07346_amd as br
V, E, M, tune = (int(x) for x in sys.argv[1:5])
e = np.random.default_rng(V).integers(0, V, size=(E, 2)).astype(np.int32)
d = torch.from_numpy(e).cuda()
ctx = br.Context(0)
ctx.set_profiling(1)
out = {}
if tune:
    out["tuned"] = ctx.autotune(d, V, M)
out["same"] = bool(np.array_equal(ctx.find(d, V, M), oracle.bridges(e, V)))
out["kind"] = int(ctx.profile()["plan_kind"])
print("RESULT " + json.dumps(out), flush=True)
""" % ROOT


def child(cache, V, E, M, tune=0):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    env = {k: v for k, v in os.environ.items() if not k.startswith("BR_")}
    r = subprocess.run([sys.executable, "-u", "-c", CHILD] + [str(x) for x in (V, E, M, tune)],
                       env=dict(env, BR_AUTOTUNE_CACHE=str(cache)), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    out = json.loads([l for l in r.stdout.splitlines() if l.startswith("RESULT ")][-1][7:])
    print(V, E, M, out, flush=True)
    assert out["same"]
    return out


def test_small_graph_entry_past_the_small_graphs(tmp_path):
    """V = 40,000 and 50,000 share an entry; "lds" 1 is the one-pass plan for both."""
    cache = tmp_path / "tune.json"
    key = child(cache, 50_000, 120_000, 8, tune=1)["tuned"]["key"]
    cache.write_text(json.dumps({key: {"lds": 1}}))
    assert child(cache, 40_000, 120_000, 8)["kind"] == 2
    assert child(cache, 50_000, 120_000, 8)["kind"] == 3
    cache.write_text(json.dumps({key: {"lds": 0, "solo": 0, "tile": 4096}}))
    assert child(cache, 50_000, 120_000, 8)["kind"] == 0       # a tree asked for by name


def test_entries_of_earlier_plans(tmp_path):
    """A file written before lists were certified in one pass (keys of five parts)
    names trees; it is neither used nor lost."""
    cache = tmp_path / "tune.json"
    key = child(cache, 50_000, 120_000, 8, tune=1)["tuned"]["key"]
    old = "|".join(key.split("|")[:5])
    cache.write_text(json.dumps({old: {"lds": 0, "solo": 1, "variant": 2}}))
    assert child(cache, 50_000, 120_000, 8)["kind"] == 3
    assert child(cache, 50_000, 120_000, 8, tune=1)["tuned"]["source"] == "measured"
    saved = json.loads(cache.read_text())
    assert saved[old] == {"lds": 0, "solo": 1, "variant": 2} and len(saved) == 2


BATCH = r"""
import sys
sys.path.insert(0, %r)
import numpy as np, torch, oracle
import paper_2108_07346_amd as br
V = 500
es = [np.random.default_rng(g).integers(0, V, size=(3000, 2)).astype(np.int32) for g in range(20)]
d = torch.from_numpy(np.concatenate(es)).cuda()
ctx = br.Context(0)
pairs, off = ctx.find_batched(d, np.arange(21, dtype=np.int64) * 3000, np.full(20, V, np.int32), 0)
assert all(np.array_equal(pairs[off[g]:off[g + 1]], oracle.bridges(e, V)) for g, e in enumerate(es))
print("CHUNK", int(ctx.profile()["rounds"]), flush=True)
""" % ROOT


def test_batch_entries_of_earlier_plans(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cache = tmp_path / "tune.json"

    def run():
        r = subprocess.run([sys.executable, "-u", "-c", BATCH], env=dict(os.environ, BR_AUTOTUNE_CACHE=str(cache)),
                           capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        return int(r.stdout.split("CHUNK")[1])

    run()
    [key] = json.loads(cache.read_text())
    old = "|".join(key.split("|")[:5])
    cache.write_text(json.dumps({old: {"chunk_edges": 1234, "blocks_per_cu": 1}}))
    assert run() != 1234
    saved = json.loads(cache.read_text())
    assert saved[old]["chunk_edges"] == 1234 and len(saved) == 2


def test_plans_are_timed_over_the_whole_query():
    """A sparse list, whose final step takes longer than its certificate: what the
    tuner reports as the winner's time is the query's (the certificate is a quarter
    of it), and ids out of range stay no error of the tuner."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import time

    import paper_2108_07346_amd as br
    V, E, M = 100_003, 200_000, 3
    e = np.random.default_rng(V).integers(0, V, size=(E, 2)).astype(np.int32)
    d = torch.from_numpy(e).cuda()
    ctx = br.Context(0)
    ms = ctx.autotune(d, V, M)["ms"]
    best = 1e30
    for _ in range(10):
        a = time.perf_counter()
        ctx.find(d, V, M)
        best = min(best, 1000 * (time.perf_counter() - a))
    print("tuner %.3f ms, query %.3f ms" % (ms, best), flush=True)
    assert ms > 0.5 * best
    e[7, 1] = V
    assert ctx.autotune(torch.from_numpy(e).cuda(), V, M + 1)["source"] == "measured"
    ctx.close()
