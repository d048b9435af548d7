"""The launch shapes that the cost rule picks for grids without a tuned entry
(no device needed): every pick is a shape its kernel supports, with a march
inside the grid, at the edges of the rule's ranges."""
import ctypes

import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")

GRIDS = [(1, 1, 1), (2, 1, 3), (7, 1000, 1), (63, 64, 65), (65, 3, 129), (129, 5, 2), (500, 500, 63), (400, 400, 100),
         (401, 400, 100), (171, 171, 171), (172, 171, 171), (1000, 1000, 64), (999, 1001, 65), (3, 3, 20000),
         (100000, 3, 3), (3, 100000, 7)]


@pytest.mark.parametrize("kind,dtypes", [("forward", ("float32", "float64", "bfloat16", "float16")),
                                         ("zfast", ("float32", "float64", "bfloat16", "float16")),
                                         ("tangent", ("float32", "float64")), ("adjoint", ("float32", "float64"))])
def test_picks_are_supported_shapes(kind, dtypes):
    try:
        lib = B.lib()
    except B.PWLibraryMissing:
        pytest.skip("library not built")
    for name in dtypes:
        dt = getattr(torch, name)
        for nx, ny, nz in GRIDS:
            t = B.launch_shape(kind, nx, ny, nz, dt)
            march = {"zfast": nx, "adjoint": nz + 2}.get(kind, nz)
            assert 1 <= t[2] <= march, (kind, name, (nx, ny, nz), t)
            if kind != "forward":
                continue
            # the entry point's own check accepts the shape: made-up device addresses pass the argument checks and
            # fail only for want of a device (or of device memory behind them)
            a, mb, n = 1 << 40, 1 << 36, ctypes.c_void_p
            c = B.pw_coeffs(0.1, 0.1, n(a + 6 * mb), n(a + 7 * mb), n(a + 8 * mb), n(a + 9 * mb))
            code = {"float32": B.PW_F32, "float64": B.PW_F64, "bfloat16": B.PW_BF16, "float16": B.PW_F16}[name]
            st = lib.pw_advect_ex(ctypes.byref(B.pw_grid(nx, ny, nz, 1)), None, code, a, a + mb, a + 2 * mb,
                                  ctypes.byref(c), a + 3 * mb, a + 4 * mb, a + 5 * mb, ctypes.byref(B.pw_tile(*t)), None)
            assert st in (B.PW_ERR_NO_DEVICE, B.PW_ERR_INVALID_ARG) and "tile" not in B.pw_last_error(), (t, st)


def test_which_boundary_gradients_read_through_the_rules():
    p = [tuple(B.HALO_MODES[m] for m in ("periodic", "copy", "zero"))] * 3
    x = [torch.zeros(5, 6, 7) for _ in range(3)]
    goes = B._bc_adjoint_reads_through
    assert goes(*x, p) and goes(*[t.double() for t in x], p)
    assert goes(*x, p[:2] + [(1, 5, 2)])                      # copy / reflect_neg, zero / copy: all nearest-cell
    for codes in (p[:2] + [(0, 2, 3)], p[:2] + [(1, 1, 3)], [(9, 9, 9)] * 3):
        assert not goes(*x, codes)
    assert not goes(*[t.bfloat16() for t in x], p)            # no such adjoint
    assert not goes(x[0], x[1], x[2].double(), p)
    assert not goes(*[torch.zeros(5, 6, 9)[:, :, :7] for _ in range(3)], p)
    assert not goes(*[torch.zeros(7, 6, 5).permute(2, 1, 0) for _ in range(3)], p)
    assert not goes(x[0], x[1], torch.zeros(5, 6, 8)[:, :, :7], p)
    assert not goes(*[torch.zeros(6, 7) for _ in range(3)], p)
