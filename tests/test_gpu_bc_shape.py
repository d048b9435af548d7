"""The launch shape of the forward under boundary rules: chosen for the plain
strips that it runs, where the forward without rules packs narrow rows."""
import os
import re
import subprocess
import sys

import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

CODE = """
import torch
from paper_2301_13016_amd import binding as B
for nx, ny, nz in {grids}:
    x = [torch.rand((nz + 2, ny + 2, nx + 2), device="cuda") for _ in range(3)]
    c = B.Coeffs(0.0025, 0.003, *[torch.rand(nz, device="cuda") for _ in range(4)])
    a = B.advect_bc(*x, c, ("periodic", "periodic", "copy"))
    B.halo_fill(x, ("periodic", "periodic", "copy"))
    b = B.advect(*x, c)
    torch.cuda.synchronize()
    assert all(torch.equal(p, q) for p, q in zip(a, b))
"""


def test_rules_have_their_own_shapes():
    grids = [(134, 95, 92), (80, 400, 120), (100, 300, 64)]
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, PWADV_LOG="1", PYTHONPATH=root)
    env.pop("PWADV_TILE", None)
    r = subprocess.run([sys.executable, "-c", CODE.format(grids=grids)], env=env, cwd=root, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    for nx, ny, nz in grids:
        m = re.search(r"pw_advect_bc %dx%dx%d halo 1 f32 tile \(([^)]*)\) default" % (nx, ny, nz), r.stderr)
        assert m, r.stderr
        assert tuple(map(int, m.group(1).split(", "))) != B.launch_shape("forward", nx, ny, nz, torch.float32)
