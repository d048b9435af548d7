"""The strips that the launch rule counts are the ones a launch runs (no device
needed): one function counts for both, compiled here with hooks around it."""
import ctypes

import pytest

import hooks
from paper_2301_13016_amd import binding as B

F32 = B.PW_F32


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    lib = hooks.load(tmp_path_factory.mktemp("hooks"))
    lib.count_strips.restype = ctypes.c_int64
    lib.count_strips.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int,
                                 ctypes.POINTER(ctypes.c_int)]
    lib.march_length.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int,
                                 ctypes.c_double, ctypes.c_int]
    lib.pick.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int,
                         ctypes.POINTER(ctypes.c_int32)]
    return lib


def count(lib, lead, rows, cols, ry, may_pack):
    packed = ctypes.c_int()
    n = lib.count_strips(lead, rows, cols, ry, may_pack, packed)
    return n, bool(packed.value)


def pick(lib, zfast, dtype, grid, rules):
    out = (ctypes.c_int32 * 6)()
    lib.pick(zfast, dtype, *grid, rules, out)
    return tuple(out)


def covered(n, blocks, pieces):
    """How often each (block, element) is stored by packed pieces, as the
    kernels number them: lanes 1..62 of the 64 positions around a piece."""
    seen = {}
    for t in range(pieces):
        for lane in range(1, 63):
            at = min(t * 62 + lane, blocks * (n + 2) - 1)
            block, i = at // (n + 2), at % (n + 2) - 1
            if 0 <= i < n:
                seen[block, i] = seen.get((block, i), 0) + 1
    return seen


@pytest.mark.parametrize("lead", [1, 2, 31, 60, 61, 62, 63, 64, 65, 66, 75, 124, 125, 126, 128, 130, 200, 310])
@pytest.mark.parametrize("rows,ry", [(1, 1), (3, 2), (4, 4), (9, 4), (17, 1)])
def test_counted_strips_cover_the_grid(shim, lead, rows, ry):
    blocks = -(-rows // ry)
    plain = -(-lead // 64) * blocks
    assert count(shim, lead, rows, 64, ry, 0) == (plain, False)
    assert count(shim, lead, rows, 128, ry, 1) == (-(-lead // 128) * blocks, False)
    n, packed = count(shim, lead, rows, 64, ry, 1)
    assert n <= plain and packed == (n < plain)
    if packed:
        seen = covered(lead, blocks, n)
        assert len(seen) == lead * blocks and set(seen.values()) == {1}
        assert len(covered(lead, blocks, n - 1)) < lead * blocks or (blocks * (lead + 2) - 2) % 62 == 0


GRIDS = [(75, 300, 100), (134, 95, 92), (100, 300, 64), (75, 300, 300), (140, 300, 150), (80, 400, 120), (40, 200, 64),
         (66, 200, 200), (42, 587, 100), (158, 229, 205), (300, 300, 75), (70, 90, 66)]


def march_cost(strips, z, march, slots, start):
    q = strips * -(-march // z) / slots
    part = q - int(q)
    return (int(q) + (max(part, 0.8) if part > 0 else 0.0)) * (z + start)


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("may_pack", [0, 1])
@pytest.mark.parametrize("ry", [1, 2, 4])
def test_the_march_is_cut_for_the_strips_that_run(shim, grid, ry, may_pack):
    """The rule's march length is the cheapest for the strips of the launch,
    packed or not, and not for another count of them."""
    nx, ny, nz = grid
    strips, _ = count(shim, nx, ny, 64, ry, may_pack)
    for slots, start in ((2048, 1.5), (1024, 0.5)):
        z = shim.march_length(nx, ny, nz, 64, ry, slots, start, may_pack)
        cuts = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16, 24, 32, 48, 64, 128, min(128, slots // strips)} - {0}
        best = min(march_cost(strips, -(-nz // c), nz, slots, start) for c in cuts if c <= nz)
        assert march_cost(strips, z, nz, slots, start) == pytest.approx(best, rel=1e-12)


def test_rules_change_the_pick(shim):
    """Narrow grids: packed strips without boundary rules, plain ones with."""
    for grid in GRIDS[:3]:
        assert pick(shim, 0, F32, grid, 0) != pick(shim, 0, F32, grid, 1) == pick(shim, 0, F32, grid, 2)
