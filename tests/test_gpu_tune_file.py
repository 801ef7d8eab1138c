"""Tuned plans whose pick comes from a cache file: the launch it names beside
the reported shape is taken and gives the reported form's grids; entries that
name shapes or forms that are not offered are tuned again."""
import json
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import sys; sys.path.insert(0, %r)
import torch
from paper_2306_13002_amd.stencil import Plan
for n in %r:
    u = torch.rand([e + 2 for e in reversed(n)], dtype=torch.float64, device='cuda',
                   generator=torch.Generator(device='cuda').manual_seed(5))
    print('START', n, file=sys.stderr, flush=True)
    with Plan('heat3d7', n, coef=(0.4, 0.1), tune='exhaustive') as p:
        cfg = p.config()
        got = [u.clone(), u.clone()]
        p.run(got, iterations=5)
    with Plan('heat3d7', n, coef=(0.4, 0.1), **cfg) as q:
        want = [u.clone(), u.clone()]
        q.run(want, iterations=5)
    print(torch.equal(got[0], want[0]), flush=True)
"""

# edits of one entry each: None leaves it
GOOD = [{"run": [7, 58, 10, 4]}, {"run": [1, 62, 14, 2]}, {}]
BAD = [{"run": [1, 62, 14, 0]}, {"run": [0, 64, 4, 1]}, {"run": [8, 5, 16, 0]}, {"run": [7, 58, 11, 4]},
       {"variant": 0, "tx": 64, "ty": 4, "zb": 1}, {"variant": 1, "tx": 32, "ty": 8, "zb": 0}, {"variant": 9}]


def plans(sizes, cache):
    env = dict(os.environ, STENCIL_TUNE_CACHE=str(cache), STENCIL_LOG="1")
    r = subprocess.run([sys.executable, "-c", CODE % (ROOT, sizes)], env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout.split(), ["tune kind=2" in part for part in r.stderr.split("START")[1:]]


def test_entries_of_a_file(tmp_path):
    cache = tmp_path / "tune.jsonl"
    edits = GOOD + BAD
    sizes = [(20 + i, 12, 9) for i in range(len(edits))]
    same, tuned = plans(sizes, cache)
    assert same == ["True"] * len(sizes) and all(tuned)
    lines = []
    for line, ed in zip(cache.read_text().splitlines(), edits):
        e = json.loads(line)
        e.update({"variant": 1, "tx": 32, "ty": 8, "zb": 4, "run": [1, 62, 14, 2]})
        e.update(ed)
        lines.append(json.dumps({k: e[k] for k in ("key", "variant", "tx", "ty", "zb", "map", "us", "run")}))
    cache.write_text("\n".join(lines) + "\n")
    same, tuned = plans(sizes, cache)
    assert same == ["True"] * len(sizes)
    assert tuned == [False] * len(GOOD) + [True] * len(BAD)
