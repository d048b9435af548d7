"""Packed strips of the z-fastest kernel (one level per lane, row blocks end to
end): columns that end inside, at and after a piece of 62 positions, row counts
that leave the last block short, against the x-fastest kernel bit for bit."""
import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64, torch.bfloat16])
@pytest.mark.parametrize("shape,halo", [((3, 1, 1), 1), ((5, 7, 1), 2), ((4, 40, 2), 1), ((6, 33, 20), 1), ((3, 9, 31), 3),
                                        ((5, 6, 59), 1), ((5, 6, 60), 1), ((5, 6, 61), 1), ((9, 13, 66), 2), ((4, 5, 75), 1),
                                        ((2, 31, 100), 1), ((3, 7, 122), 1), ((3, 7, 130), 1), ((2, 5, 186), 1)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else "h%d" % s)
def test_bits_of_the_x_fastest_kernel(shape, halo, dtype):
    nx, ny, nz = shape
    odt = torch.float64 if dtype == torch.float64 else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx + 100 * ny + 10000 * nz)
    x = [(torch.rand((nz + 2 * halo, ny + 2 * halo, nx + 2 * halo), device="cuda", generator=gen) - 0.5).to(dtype)
         for _ in range(3)]
    add = [torch.rand((nz, ny, nx), device="cuda", generator=gen).to(odt) for _ in range(3)]
    c = B.Coeffs(0.25, 0.5, *[torch.rand(nz, device="cuda", generator=gen).to(odt) for _ in range(4)])
    want = B.advect(*x, c, halo=halo)
    want_e = B.advect_epilogue(*x, c, add, alpha=0.75, halo=halo)
    xz = [t.permute(2, 1, 0).contiguous() for t in x]
    az = [torch.empty((nx, ny, nz), device="cuda", dtype=odt).copy_(t.permute(2, 1, 0)) for t in add]
    for tile in (None, (1, 1, 2, 1), (1, 2, 64, 4), (1, 2, 3, 8, 2), (1, 4, 1, 4), (1, 4, 5, 1, 2), (1, 8, 2, 2)):
        if tile is not None and tile[2] > nx:
            tile = tile[:2] + (nx,) + tile[3:]
        got = [torch.full((nx, ny, nz), float("nan"), device="cuda", dtype=odt) for _ in range(3)]
        B.advect_zfast(*xz, c, halo=halo, out=got, tile=tile)
        got_e = [torch.full((nx, ny, nz), float("nan"), device="cuda", dtype=odt) for _ in range(3)]
        B.advect_zfast_epilogue(*xz, c, az, alpha=0.75, halo=halo, out=got_e, tile=tile)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a.permute(2, 1, 0), b), (shape, tile)
        for a, b in zip(got_e, want_e):
            assert torch.equal(a.permute(2, 1, 0), b), (shape, tile)
