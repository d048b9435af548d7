"""Packed strips of the forward kernel (one column per lane, row blocks end to
end): widths that end inside, at and after a piece of 62 positions, row counts
that leave the last block short, against strips of wider lanes bit for bit,
with nothing written outside the outputs."""
import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

SHAPES = [(8, 1, 1), (9, 40, 2), (20, 33, 6), (31, 9, 3), (58, 6, 5), (59, 6, 5), (60, 6, 5), (61, 6, 5), (66, 13, 9),
          (75, 5, 4), (100, 31, 2), (122, 7, 3), (124, 7, 3), (130, 7, 3), (186, 5, 2), (248, 3, 2)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("halo", [1, 3])
def test_bits_of_wider_lanes(dtype, halo):
    odt = torch.float64 if dtype == torch.float64 else torch.float32
    wide = (2, 2) if dtype == torch.float64 else (4, 2)
    for nx, ny, nz in SHAPES:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(nx + 100 * ny + 10000 * nz)
        x = [(torch.rand((nz + 2 * halo, ny + 2 * halo, nx + 2 * halo), device="cuda", generator=gen) - 0.5).to(dtype)
             for _ in range(3)]
        add = [torch.rand((nz, ny, nx), device="cuda", generator=gen).to(odt) for _ in range(3)]
        c = B.Coeffs(0.25, 0.5, *[torch.rand(nz, device="cuda", generator=gen).to(odt) for _ in range(4)])
        want = B.advect(*x, c, halo=halo, tile=(*wide, nz, 1))
        want_e = B.advect_epilogue(*x, c, add, alpha=0.75, halo=halo, tile=(*wide, nz, 1))
        inner = [t[halo:-halo, halo:-halo, halo:-halo] for t in x]
        n = nx * ny * nz
        for ry, z, w, depth in ((1, 1, 4, 1), (1, nz, 1, 2), (2, max(1, nz // 2), 8, 1), (2, nz, 4, 2), (4, 1, 1, 1), (4, nz, 2, 2)):
            bufs = [torch.full((n + 256,), 7.25, dtype=odt, device="cuda") for _ in range(6)]
            outs = [b[128:128 + n].view(nz, ny, nx) for b in bufs]
            B.advect(*x, c, halo=halo, tile=(1, ry, z, w, depth), out=outs[:3])
            B.advect_epilogue(*x, c, add, alpha=0.75, halo=halo, tile=(1, ry, z, w, depth), out=outs[3:])
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(outs, [*want, *want_e])), (nx, ny, nz, ry, z, w, depth)
            assert all(bool((b[:128] == 7.25).all()) and bool((b[-128:] == 7.25).all()) for b in bufs)
            if dtype == odt:   # addends that are the fields' own interiors, output in their layout
                nxt = [t.clone() for t in x]
                ni = [t[halo:-halo, halo:-halo, halo:-halo] for t in nxt]
                B.advect_epilogue(*x, c, inner, alpha=0.5, halo=halo, tile=(1, ry, z, w, depth), out=ni)
                ref = B.advect_epilogue(*x, c, [t.contiguous() for t in inner], alpha=0.5, halo=halo, tile=(*wide, nz, 1))
                torch.cuda.synchronize()
                assert all(torch.equal(a, b) for a, b in zip(ni, ref)), (nx, ny, nz, ry, z, w, depth)
