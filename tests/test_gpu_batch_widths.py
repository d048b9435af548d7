"""The batched form where each subdomain has strips of its own width: one, two
and four columns per lane at the widths where the choice changes, bit for bit
the single-grid results, and the work list that the rule gives."""
import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

SHAPES = [(1, 3, 2), (63, 5, 33), (64, 4, 40), (65, 9, 3), (127, 2, 7), (128, 6, 31), (129, 3, 32), (255, 5, 9),
          (256, 4, 17), (257, 3, 5), (300, 2, 34), (515, 1, 3)]


@pytest.mark.parametrize("tile", [None, (0, 4, 32, 4), (0, 4, 7, 1, 2), (0, 4, 16, 8)])
def test_each_width_equals_single_grid(tile):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(31)
    subs = []
    for nx, ny, nz in SHAPES:
        x = [torch.rand((nz + 2, ny + 2, nx + 2), device="cuda", generator=gen) - 0.5 for _ in range(3)]
        c = B.Coeffs(0.25, 0.5, *[torch.rand(nz, device="cuda", generator=gen) for _ in range(4)])
        subs.append((*x, c, tuple(torch.full((nz, ny, nx), float("nan"), device="cuda") for _ in range(3))))
    b = B.Batch(subs, tile=tile)
    used, items, _ = b.info()
    if used[0] == 0 and used[1] == 4:
        want = 0
        for nx, ny, nz in SHAPES:
            px = 1 if nx <= 64 else 2 if nx <= 128 else 4
            zl = -(-nz // -(-nz // used[2]))
            want += -(-nx // (64 * px)) * -(-ny // (2 if px == 4 else 4)) * -(-nz // zl)
        assert items == want
    b.run()
    torch.cuda.synchronize()
    for (u, v, w, c, got), s in zip(subs, SHAPES):
        for a, r in zip(got, B.advect(u, v, w, c)):
            assert torch.equal(a, r), s
    b.close()
