"""How the last round of an FFN launch is cut, on the CPU: the cut that the
re-batch chooses is the cheapest of all that are possible, where a cut's cost
is the largest sum that any workgroup gets -- not that of a sample of
workgroups, under which a family can lie between the samples, count as free
and be left whole."""

import ctypes
import itertools

import numpy as np
import pytest

import ffn_host

SPLIT_BYTES = 128 * 256 * 256 * 4
NWG = 256


@pytest.fixture(scope="module")
def lib():
    so = ffn_host.load()
    so.ffn_cut.argtypes = [ctypes.c_int] * 5 + [ctypes.c_long]
    so.ffn_cut_cost.argtypes = [ctypes.c_int] * 5 + [ctypes.c_long, ctypes.c_int]
    so.ffn_cut_cost.restype = ctypes.c_long
    return so


def _check(lib, tiles, kt, nwg=NWG, split_bytes=SPLIT_BYTES):
    got = lib.ffn_cut(*tiles, nwg, kt, split_bytes)
    cost = {a | b << 4 | c << 8: lib.ffn_cut_cost(*tiles, nwg, kt, split_bytes, a | b << 4 | c << 8)
            for a, b, c in itertools.product(range(1, 9), repeat=3)}
    possible = {n: v for n, v in cost.items() if v >= 0}
    total = sum(tiles)
    if total % nwg == 0 or total // nwg >= 8 or kt < 16:
        assert got == 0x111, (tiles, kt)
        return
    assert got in possible, (tiles, kt, hex(got))
    assert possible[got] == min(possible.values()), (tiles, kt, hex(got))


@pytest.mark.parametrize("tiles,kt", [
    # one expert of 340, 300 and 600 rows, d = 4096, f = 14336: its down launch
    ((16, 16, 0), 224), ((16, 0, 16), 224), ((32, 16, 0), 224),
    # eight experts of 111 .. 235 rows, d = 4096, f = 2048
    ((96, 32, 0), 64), ((96, 32, 0), 32),
    # a 4096-token layer's down launch, and one tile of each family
    ((528, 16, 16), 224), ((1, 1, 1), 64), ((255, 0, 0), 64), ((0, 1, 256), 17),
])
def test_cut_is_the_cheapest(lib, tiles, kt):
    _check(lib, tiles, kt)


def test_random_cuts_are_the_cheapest(lib):
    g = np.random.default_rng(7)
    for _ in range(300):
        nwg = int(g.choice([8, 32, 256, 304]))
        tiles = [int(g.integers(0, m)) if g.random() < 0.7 else 0 for m in (2 * nwg, nwg, nwg)]
        split_bytes = SPLIT_BYTES if g.random() < 0.7 else SPLIT_BYTES // 16
        if sum(tiles):
            _check(lib, tiles, int(np.exp(g.uniform(np.log(8), np.log(260)))), nwg, split_bytes)
