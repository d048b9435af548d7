"""GPU tests of the strips at the x end (z end in the z-fastest layout), whose
vector loads run past the row and whose stores end inside it: every launch
shape against one-column lanes, bit for bit, at widths around the lanes' and
strips' vector widths -- with dense arrays, so that the last rows of the last
plane end the allocation -- for the plain forward, the epilogue, boundary
rules and the tangent, and that nothing outside the outputs is written.
"""
import sys

import numpy as np
import pytest

from gpu_util import dev_grid
from paper_2301_13016_amd import binding as B
from paper_2301_13016_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

LID = [("periodic", "copy", "copy")] * 2 + [("periodic", "copy", "zero")]
KEEPX = [("keep", "reflect_neg", "periodic")] * 3
WIDTHS = [1, 3, 5, 8, 63, 65, 127, 130, 255, 257, 511, 515]


@pytest.fixture(autouse=True)
def _announce(request):
    sys.__stderr__.write("\n[gpu-test] %s\n" % request.node.nodeid)
    sys.__stderr__.flush()
    yield


def _guarded(shape, dtype):
    """Three output views inside larger buffers filled with a marker."""
    n = int(np.prod(shape))
    bufs = [torch.full((n + 512,), 7.25, dtype=dtype, device="cuda") for _ in range(3)]
    return bufs, tuple(b[256:256 + n].view(shape) for b in bufs)


def _untouched(bufs):
    return all(bool((b[:256] == 7.25).all()) and bool((b[-256:] == 7.25).all()) for b in bufs)


def _same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("storage", [None, "float64", "bfloat16", "float16"])
@pytest.mark.parametrize("nx", WIDTHS)
def test_forward_shapes_at_the_x_end(nx, storage):
    ny, nz = 7, 5
    g = wl.make_grid(nx, ny, nz, seed=1300 + nx, dtype=np.float64 if storage == "float64" else np.float32)
    f, c = dev_grid(g, storage=None if storage in (None, "float64") else getattr(torch, storage))
    odt = torch.float64 if storage == "float64" else torch.float32
    half = storage in ("bfloat16", "float16")
    tiles = [(2, 1, 5, 1, 1, 0), (2, 4, 3, 4, 2, 0)]
    if storage == "float64":
        tiles += [(2, 2, 3, 4, 1, 2), (2, 4, 5, 2, 1, 1)]
    else:
        tiles += [(4, 2, 2, 1, 1, 0), (4, 2, 5, 4, 1, 2), (4, 4, 3, 2, 1, 1)]
    if half:
        tiles += [(8, 1, 5, 1, 1, 0), (8, 2, 3, 4, 1, 2)]
    add = [torch.rand((nz, ny, nx), dtype=odt, device="cuda") for _ in range(3)]
    one = (1, 1, 2, 1, 1, 0)
    plain = B.advect(*f, c, tile=one)
    epi = B.advect_epilogue(*f, c, add, alpha=0.5, tile=one)
    rules = [B.advect_bc(*f, c, bc, tile=one) for bc in (LID, KEEPX)]
    both = B.advect_bc(*f, c, LID, addends=add, alpha=0.5, tile=one)
    for t in tiles:
        bufs, out = _guarded((nz, ny, nx), odt)
        assert _same(B.advect(*f, c, out=out, tile=t), plain), t
        assert _untouched(bufs), t
        assert _same(B.advect_epilogue(*f, c, add, alpha=0.5, out=out, tile=t), epi), t
        acc = tuple(x.clone() for x in add)   # in place
        assert _same(B.advect_epilogue(*f, c, acc, alpha=0.5, out=acc, tile=t), epi), t
        for bc, ref in zip((LID, KEEPX), rules):
            assert _same(B.advect_bc(*f, c, bc, out=out, tile=t), ref), (t, bc)
        assert _same(B.advect_bc(*f, c, LID, addends=add, alpha=0.5, out=out, tile=t), both), t
        assert _untouched(bufs), t


@pytest.mark.parametrize("halo", [1, 2])
@pytest.mark.parametrize("nz", [1, 3, 5, 63, 75, 129, 257])
def test_zfast_shapes_at_the_column_end(nz, halo):
    nx, ny = 6, 5
    g = wl.make_grid(nx, ny, nz, seed=1400 + nz, halo=halo)
    f, c = dev_grid(g)
    z = [x.permute(2, 1, 0).contiguous() for x in f]
    add = [torch.rand((nx, ny, nz), device="cuda") for _ in range(3)]
    one = (1, 1, 3, 1, 1, 0)
    plain = B.advect_zfast(*z, c, halo=halo, tile=one)
    epi = B.advect_zfast_epilogue(*z, c, add, alpha=0.5, halo=halo, tile=one)
    assert _same([x.permute(2, 1, 0) for x in plain], B.advect(*f, c, halo=halo, tile=(1, 1, 2, 1, 1, 0)))
    for t in [(2, 1, 6, 1, 1, 0), (2, 4, 3, 4, 2, 0), (4, 1, 2, 1, 1, 0), (4, 2, 6, 2, 2, 0)]:
        bufs, out = _guarded((nx, ny, nz), torch.float32)
        assert _same(B.advect_zfast(*z, c, halo=halo, out=out, tile=t), plain), t
        assert _same(B.advect_zfast_epilogue(*z, c, add, alpha=0.5, halo=halo, out=out, tile=t), epi), t
        assert _untouched(bufs), t


@pytest.mark.parametrize("nx", [1, 3, 64, 127, 129, 255])
def test_tangent_two_columns_at_the_x_end(nx):
    g = wl.make_grid(nx, 5, 4, seed=1500 + nx)
    f, c = dev_grid(g)
    d = [torch.from_numpy(x).cuda() for x in wl.direction(nx, 5, 4, seed=1501, dtype=np.float32)]
    ref = B.advect_tangent(*f, c, *d, tile=(1, 1, 4, 1, 1, 0))
    for t in [(2, 1, 4, 1, 1, 0), (2, 2, 3, 4, 2, 0)]:
        bufs, out = _guarded((4, 5, nx), torch.float32)
        assert _same(B.advect_tangent(*f, c, *d, out=out, tile=t), ref), t
        assert _untouched(bufs), t
