"""The one-launch fold of one-layer halos on the smallest extents, where both
halo cells of an axis may end in the same cell, against the oracle (integer
gradients: every sum is exact)."""
import itertools

import numpy as np
import pytest

from oracle import halo as H
from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

RULES = ("keep", "periodic", "copy", "zero", "reflect", "reflect_neg")


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 1, 3), (1, 3, 2), (3, 2, 1), (66, 4, 5), (3, 65, 2), (2, 2, 70)],
                         ids=lambda s: "x".join(map(str, s)))
def test_small_extents_every_rule(shape, dtype):
    nx, ny, nz = shape
    rng = np.random.default_rng(nx * 10000 + ny * 100 + nz)
    combos = list(itertools.product(RULES, repeat=3))
    for at in range(0, len(combos), 8):          # up to eight fields of different rules in one call
        modes = combos[at:at + 8]
        g = [rng.integers(-50, 50, (nz + 2, ny + 2, nx + 2)).astype(np.float64) for _ in modes]
        dev = [torch.from_numpy(x).to("cuda", dtype) for x in g]
        B.halo_fold(dev, modes)
        torch.cuda.synchronize()
        for d, x, m in zip(dev, g, modes):
            assert np.array_equal(d.cpu().to(torch.float64).numpy(), H.fold(x, 1, m)), (shape, m)
