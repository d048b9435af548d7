"""The adjoint's tile order on grids two strips wide (z-chunk fastest where the
second strip is light): gradients equal those of a march in one piece, where the
order does not matter, and coefficient gradients those in FP64, on whole numbers
that every sum holds exactly."""
import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("nx", [60, 61, 99, 100, 122, 123])   # 1 strip; 2 with 1, 39, 40 and 62 columns; 3
@pytest.mark.parametrize("halo", [1, 2])
def test_two_strips(nx, halo):
    ny, nz = 21, 23
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx + halo)
    ints = lambda s, m: torch.randint(-m, m + 1, s, device="cuda", generator=gen).float()  # noqa: E731
    x = [ints((nz + 2 * halo, ny + 2 * halo, nx + 2 * halo), 3) for _ in range(3)]
    r = [ints((nz, ny, nx), 2) for _ in range(3)]
    c = B.Coeffs(0.5, 0.25, *[ints((nz,), 2) for _ in range(4)])
    want = B.advect_adjoint(*x, c, *r, halo=halo, tile=(1, 2, nz + 2 * halo, 1, 1, 0))
    d = [t.double() for t in x], [t.double() for t in r]
    exact = B.advect_coeff_grad(*d[0], *d[1], halo=halo)
    for tile in (None, (1, 4, 3, 1, 1, 0), (1, 1, 5, 4, 2, 0), (1, 2, 1, 3, 1, 0)):
        got = B.advect_adjoint(*x, c, *r, halo=halo, tile=tile)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want)), tile
    both, grads = B.advect_adjoint_coeff_grad(*x, c, *r, halo=halo)
    alone = B.advect_coeff_grad(*x, *r, halo=halo)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(both, want))
    for name in exact:
        assert torch.equal(grads[name], exact[name]) and torch.equal(alone[name], exact[name]), name
