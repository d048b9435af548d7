"""Four-row shared shapes on grids of whole strips in x, which run kernels of
their own, against one-column strips bit for bit (and one column more, which
does not take them)."""
import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("strips,more,ny,nz", [(1, 0, 1, 1), (1, 0, 17, 5), (2, 0, 33, 9), (1, 1, 17, 5)])
def test_bits_of_one_column_strips(dtype, strips, more, ny, nz):
    odt = torch.float64 if dtype == torch.float64 else torch.float32
    px = 2 if dtype == torch.float64 else 4
    nx = strips * 64 * px + more
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx + ny)
    x = [(torch.rand((nz + 2, ny + 2, nx + 2), device="cuda", generator=gen) - 0.5).to(dtype) for _ in range(3)]
    c = B.Coeffs(0.25, 0.5, *[torch.rand(nz, device="cuda", generator=gen).to(odt) for _ in range(4)])
    want = B.advect(*x, c, tile=(1, 2, nz, 1))
    for z in {1, (nz + 1) // 2, nz}:
        for w in (2, 4):
            for share in (1, 2):
                bufs = [torch.full((nx * ny * nz + 256,), 7.25, dtype=odt, device="cuda") for _ in range(3)]
                out = [b[128:-128].view(nz, ny, nx) for b in bufs]
                B.advect(*x, c, tile=(px, 4, z, w, 1, share), out=out)
                torch.cuda.synchronize()
                assert all(torch.equal(a, b) for a, b in zip(out, want)), (z, w, share)
                assert all(bool((b[:128] == 7.25).all()) and bool((b[-128:] == 7.25).all()) for b in bufs)
