"""Gradients through the boundary rules: values read through the rules against
filled copies, bit for bit (the same numbers meet the same arithmetic), at the
edges of strips, on the smallest extents, for every kind of rule."""
import random

import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

NEAREST = ("copy", "zero", "reflect", "reflect_neg")


def through_copies(x, c, bc, r, halo):
    filled = [t.clone() for t in x]
    B.halo_fill(filled, bc, halo=halo)
    return B.halo_fold(list(B.advect_adjoint(*filled, c, *r, halo=halo)), bc, halo=halo)


def bits(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int64)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shape,halo", [((1, 1, 1), 1), ((2, 1, 3), 1), ((5, 3, 2), 2), ((60, 6, 4), 1), ((61, 7, 5), 1),
                                        ((59, 5, 9), 2), ((124, 4, 3), 1), ((130, 9, 6), 3), ((200, 33, 40), 1)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else "h%d" % s)
def test_bits_of_filled_copies(shape, halo, dtype):
    nx, ny, nz = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx + 7 * ny + 31 * nz + halo)
    rng = random.Random(nx * ny + nz)
    mk = lambda s: (torch.rand(s, device="cuda", generator=gen) * 20 - 10).to(dtype)  # noqa: E731
    x = [mk((nz + 2 * halo, ny + 2 * halo, nx + 2 * halo)) for _ in range(3)]
    r = [mk((nz, ny, nx)) for _ in range(3)]
    c = B.Coeffs(0.0025, 0.003, *[mk((nz,)) for _ in range(4)])
    n = {"x": nx, "y": ny, "z": nz}
    for _ in range(12):
        axes = []
        for d in "xyz":
            kind = rng.choice(["keep", "periodic", "nearest", "nearest"])
            rules = [m for m in NEAREST if n[d] >= halo or not m.startswith("reflect")]
            axes.append([kind] * 3 if kind != "nearest" else [rng.choice(rules) for _ in range(3)])
        bc = list(zip(*axes))
        want = through_copies(x, c, bc, r, halo)
        got = B.advect_bc_adjoint(*x, c, bc, *r, halo=halo)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(bits(a), bits(b)), (shape, halo, bc)


def test_halo_under_other_rules_is_not_read():
    """NaN in the halo of axes whose rule is not keep stays out of the
    gradients, and the winds are left as they were."""
    nx, ny, nz, bc = 70, 9, 6, ("periodic", "copy", "reflect_neg")
    x = [torch.rand((nz + 2, ny + 2, nx + 2), device="cuda") for _ in range(3)]
    r = [torch.rand((nz, ny, nx), device="cuda") for _ in range(3)]
    c = B.Coeffs(0.0025, 0.003, *[torch.rand(nz, device="cuda") for _ in range(4)])
    want = through_copies(x, c, bc, r, 1)
    for t in x:
        inner = t[1:-1, 1:-1, 1:-1].clone()
        t.fill_(float("nan"))
        t[1:-1, 1:-1, 1:-1] = inner
    before = [t.clone() for t in x]
    got = B.advect_bc_adjoint(*x, c, bc, *r)
    torch.cuda.synchronize()
    assert all(torch.equal(bits(a), bits(b)) for a, b in zip(got, want))
    assert all(torch.equal(bits(a), bits(b)) for a, b in zip(x, before))


def test_calls_that_go_through_copies_still_do():
    """Strided winds and rules of different kinds on one axis."""
    nx, ny, nz = 20, 6, 5
    r = [torch.rand((nz, ny, nx), device="cuda") for _ in range(3)]
    c = B.Coeffs(0.0025, 0.003, *[torch.rand(nz, device="cuda") for _ in range(4)])
    x = [torch.rand((nz + 2, ny + 2, nx + 2), device="cuda") for _ in range(3)]
    views = [torch.zeros((nz + 3, ny + 2, nx + 9), device="cuda")[:nz + 2, :, :nx + 2].copy_(t) for t in x]
    for winds, bc in [(views, ("periodic", "periodic", "copy")),
                      (x, [("periodic", "copy", "copy"), ("copy", "copy", "copy"), ("keep", "copy", "zero")])]:
        want = through_copies(x, c, bc, r, 1)
        got = B.advect_bc_adjoint(*winds, c, bc, *r)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want)), bc
