"""Argument checks of pw_advect_bc_adjoint (no device needed): made-up device
addresses pass them and fail only for want of a device."""
import ctypes

import pytest

from paper_2301_13016_amd import binding as B

A, MB, P = 1 << 40, 1 << 28, ctypes.c_void_p
KEEP, PERIODIC, COPY, ZERO, REFLECT, NEG = (B.HALO_MODES[m] for m in ("keep", "periodic", "copy", "zero", "reflect",
                                                                      "reflect_neg"))


def call(rules=((PERIODIC, PERIODIC, COPY),) * 3, dtype=B.PW_F32, grid=(20, 6, 5, 1), tile=None, layout=None, at=None,
         no_rules=False):
    """Status of a call on nine arrays of their own, some moved by ``at`` (name -> address)."""
    names = ("u", "v", "w", "gsu", "gsv", "gsw", "gu", "gv", "gw", "c")
    p = {n: A + i * MB for i, n in enumerate(names)}
    p.update(at or {})
    c = B.pw_coeffs(0.1, 0.1, *(P(p["c"] + i * 4096) for i in range(4)))
    modes = None if no_rules else (B.pw_halo_modes * 3)(*(B.pw_halo_modes(*r) for r in rules))
    return B.lib().pw_advect_bc_adjoint(B.pw_grid(*grid), layout, dtype, *(p[n] for n in names[:3]), c, modes,
                                        *(p[n] for n in names[3:9]), tile, None)


@pytest.fixture(autouse=True)
def built():
    try:
        B.lib()
    except B.PWLibraryMissing:
        pytest.skip("library not built")


def test_good_arguments_reach_the_device():
    for rules in (((PERIODIC, PERIODIC, COPY),) * 3, ((KEEP, KEEP, KEEP),) * 3,
                  ((COPY, ZERO, REFLECT), (NEG, REFLECT, ZERO), (ZERO, COPY, NEG))):
        for dtype in (B.PW_F32, B.PW_F64):
            for tile in (None, B.pw_tile(1, 4, 3, 8, 2, 0)):
                st = call(rules, dtype, tile=tile)
                assert st == B.PW_ERR_NO_DEVICE or "device" in B.pw_last_error(), B.pw_last_error()


@pytest.mark.parametrize("kw,status", [
    (dict(no_rules=True), B.PW_ERR_INVALID_ARG),
    (dict(rules=((9, 1, 1),) * 3), B.PW_ERR_INVALID_ARG),
    (dict(rules=((PERIODIC, COPY, COPY), (COPY, COPY, COPY), (COPY, COPY, COPY))), B.PW_ERR_UNSUPPORTED),
    (dict(rules=((COPY, COPY, COPY), (COPY, COPY, COPY), (COPY, COPY, KEEP))), B.PW_ERR_UNSUPPORTED),
    (dict(rules=((REFLECT, COPY, COPY),) * 3, grid=(2, 6, 5, 3)), B.PW_ERR_INVALID_ARG),
    (dict(dtype=B.PW_BF16), B.PW_ERR_UNSUPPORTED),
    (dict(dtype=B.PW_F16), B.PW_ERR_UNSUPPORTED),
    (dict(dtype=17), B.PW_ERR_INVALID_ARG),
    (dict(grid=(0, 6, 5, 1)), B.PW_ERR_INVALID_ARG),
    (dict(tile=B.pw_tile(2, 2, 4, 1, 1, 0)), B.PW_ERR_INVALID_ARG),
    (dict(tile=B.pw_tile(1, 3, 4, 1, 1, 0)), B.PW_ERR_INVALID_ARG),
    (dict(at={"gu": None}), B.PW_ERR_INVALID_ARG),
    (dict(at={"gu": A + 6 * MB + 2}), B.PW_ERR_INVALID_ARG),
    (dict(at={"gu": A}), B.PW_ERR_INVALID_ARG),              # on u
    (dict(at={"gv": A + 6 * MB + 64}), B.PW_ERR_INVALID_ARG),  # on gu
    (dict(at={"gw": A + 3 * MB}), B.PW_ERR_INVALID_ARG),      # on gsu
    (dict(at={"gw": A + 9 * MB}), B.PW_ERR_INVALID_ARG),      # on the coefficients
    (dict(layout=B.pw_layout(21, 22 * 8, 20, 120)), B.PW_ERR_INVALID_ARG),
])
def test_bad_arguments_are_refused_before_any_device_work(kw, status):
    assert call(**kw) == status and "device" not in B.pw_last_error(), B.pw_last_error()
