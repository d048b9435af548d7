"""The shapes that tuning a batch times (no device needed): the one the batch has
first, every length that a batch gets by default among them, none twice."""
import ctypes

import pytest

import hooks


@pytest.fixture(scope="module")
def candidates(tmp_path_factory):
    lib = hooks.load(tmp_path_factory.mktemp("hooks"))
    tile = ctypes.c_int32 * 6
    lib.batch_candidates.argtypes = [tile, tile * 512, ctypes.c_int]

    def get(*start):
        out = (tile * 512)()
        n = lib.batch_candidates(tile(*start), out, 512)
        return [tuple(t) for t in out[:n]]
    return get


@pytest.mark.parametrize("start", [(0, 4, 16, 4, 1, 0), (0, 4, 32, 4, 1, 0), (4, 2, 64, 4, 2, 0), (1, 2, 19, 3, 1, 0)])
def test_start_and_default_lengths_are_timed(candidates, start):
    c = candidates(*start)
    assert c[0] == start
    assert len(set(c)) == len(c) > 100
    for zlen in (16, 32, 64):
        assert (0, 4, zlen, 4, 1, 0) in c
