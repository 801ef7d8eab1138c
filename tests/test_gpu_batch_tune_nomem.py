"""A batch class whose tuning finds no room for scratch grids takes the launch
of its largest problem's own tuning (here from a cache file, a launch that the
defaults would not take).  The grids described are larger than any card, so
nothing is run: the plan logs what it launches."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
N = (128, 64, 1 << 24)  # 1.15 TB per grid

CODE = """
import sys; sys.path.insert(0, %r)
from paper_2306_13002_amd.stencil import BatchPlan, Plan
if sys.argv[1] == 'single':
    Plan('heat3d7', (20, 12, 9), coef=(0.4, 0.1), variant='saturated_t2', tune='exhaustive', tile_map='natural').close()
else:
    BatchPlan([%r], coef=(0.4, 0.1), variant='saturated_t2', tune='exhaustive').close()
"""


def call(what, cache):
    env = dict(os.environ, STENCIL_TUNE_CACHE=str(cache), STENCIL_LOG="1")
    r = subprocess.run([sys.executable, "-c", CODE % (ROOT, N), what], env=env, capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    return r


def test_launch_of_the_largest_problems_tuning(tmp_path):
    cache = tmp_path / "tune.jsonl"
    call("single", cache)
    e = json.loads(cache.read_text())
    dims = lambda n: "n%dx%dx%d/r1/py%d/pz%d/" % (*n, n[0] + 2, (n[0] + 2) * (n[1] + 2))  # noqa: E731
    assert dims((20, 12, 9)) in e["key"]
    e["key"] = e["key"].replace(dims((20, 12, 9)), dims(N))
    e.update(tx=32, ty=8, zb=1 << 22, run=[6, 60, 12, 1 << 22])
    cache.write_text(json.dumps({k: e[k] for k in ("key", "variant", "tx", "ty", "zb", "map", "us", "run")}) + "\n")
    r = call("batch", cache)
    assert "on its largest problem alone" in r.stderr
    assert "variant=6 tile=(60,12,4194304) items=72" in r.stderr, r.stderr[-1500:]
