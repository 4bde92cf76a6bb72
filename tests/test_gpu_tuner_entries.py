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
