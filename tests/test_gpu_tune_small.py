"""Tuning does not leave a grid slower than the shape that untuned calls take,
where that is none of the tuner's own candidates (a small grid's march cut into
single levels)."""
import os
import subprocess
import sys

import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

GRID = """
import torch
from paper_2301_13016_amd import binding as B
nx, ny, nz = 32, 32, 64
before = B.launch_shape("forward", nx, ny, nz, torch.float32)
after = B.tune(nx, ny, nz, torch.float32, flags=1)[0]   # the forward only
s = torch.cuda.Stream()
x = [torch.rand((nz + 2, ny + 2, nx + 2), device="cuda") for _ in range(3)]
o = [torch.empty((nz, ny, nx), device="cuda") for _ in range(3)]
c = B.Coeffs(0.0025, 0.003, *[torch.rand(nz, device="cuda") for _ in range(4)])
def graph(tile):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        for _ in range(200):
            B.advect(*x, c, out=o, tile=tile, stream=s)
    return g
def us(g):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    with torch.cuda.stream(s):
        a.record(s); g.replay(); b.record(s)
    b.synchronize()
    return a.elapsed_time(b) * 5
B.advect(*x, c, out=o, tile=before, stream=s)
torch.cuda.synchronize()
ga, gb = graph(after), graph(before)
t = [(us(ga), us(gb)) for _ in range(9)][2:]
print(before, after, min(p for p, _ in t), min(q for _, q in t))
assert min(p for p, _ in t) <= 1.15 * min(q for _, q in t)
"""


def test_a_small_grid():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, PYTHONPATH=root)   # a process of its own: the tuning table is process-wide
    for name in ("PWADV_TILE", "PWADV_TUNE_CACHE"):
        env.pop(name, None)
    r = subprocess.run([sys.executable, "-c", GRID], env=env, cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
