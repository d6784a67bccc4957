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
    so.ffn_cut.argtypes = [ctypes.c_int] * 6 + [ctypes.c_long]
    so.ffn_cut_cost.argtypes = [ctypes.c_int] * 6 + [ctypes.c_long, ctypes.c_int]
    so.ffn_cut_cost.restype = ctypes.c_long
    return so


def _check(lib, fp8, tiles, kt, nwg=NWG, split_bytes=SPLIT_BYTES):
    got = lib.ffn_cut(fp8, *tiles, nwg, kt, split_bytes)
    cost = {a | b << 4 | c << 8: lib.ffn_cut_cost(fp8, *tiles, nwg, kt, split_bytes, a | b << 4 | c << 8)
            for a, b, c in itertools.product(range(1, 9), repeat=3)}
    possible = {n: v for n, v in cost.items() if v >= 0}
    total = sum(tiles)
    if total % nwg == 0 or total // nwg >= 8 or kt < 16:
        assert got == 0x111, (tiles, kt)
        return
    assert got in possible, (tiles, kt, hex(got))
    assert possible[got] == min(possible.values()), (tiles, kt, hex(got))


@pytest.mark.parametrize("fp8", [0, 1])
@pytest.mark.parametrize("tiles,kt", [
    # one expert of 340, 300 and 600 rows, d = 4096, f = 14336: its down launch
    ((16, 16, 0), 224), ((16, 0, 16), 224), ((32, 16, 0), 224),
    # eight experts of 111 .. 235 rows, d = 4096, f = 2048
    ((96, 32, 0), 64), ((96, 32, 0), 32),
    # a 4096-token layer's down launch, and one tile of each family
    ((528, 16, 16), 224), ((1, 1, 1), 64), ((255, 0, 0), 64), ((0, 1, 256), 17),
])
def test_cut_is_the_cheapest(lib, fp8, tiles, kt):
    _check(lib, fp8, tiles, kt)


def test_random_cuts_are_the_cheapest(lib):
    g = np.random.default_rng(7)
    for i in range(300):
        nwg = int(g.choice([8, 32, 256, 304]))
        tiles = [int(g.integers(0, m)) if g.random() < 0.7 else 0 for m in (2 * nwg, nwg, nwg)]
        split_bytes = SPLIT_BYTES if g.random() < 0.7 else SPLIT_BYTES // 16
        if sum(tiles):
            _check(lib, i % 2, tiles, int(np.exp(g.uniform(np.log(8), np.log(260)))), nwg, split_bytes)


# Measured times (us, weights in HBM) of launches under cuts worth having,
# pieces of the 256-, 128- and 64-row tiles as digits: the two weight formats
# want different ones.
MEASURED = [
    # 10 experts of 40 .. 500 rows, d = 4096, f = 2048: gate/up, down
    (0, (80, 64, 48), 64, {111: 98.5, 112: 104.5, 215: 109.3, 221: 120.4, 211: 127.9}),
    (1, (80, 64, 48), 64, {111: 105.7, 112: 107.8, 215: 95.3, 214: 95.3, 221: 100.3, 211: 102.2}),
    (0, (80, 64, 48), 32, {111: 59.0, 112: 62.0, 122: 62.8, 211: 69.8, 212: 71.3}),
    (1, (80, 64, 48), 32, {111: 64.0, 112: 65.9, 122: 67.2, 211: 64.1, 212: 68.0}),
    # d = 4096, f = 14336, 400 tokens of 8 experts, top-2: down
    (0, (32, 32, 80), 224, {223: 221.9, 233: 219.9, 224: 226.5, 323: 250.6, 221: 231.5, 321: 249.6, 111: 311.2}),
    (1, (32, 32, 80), 224, {223: 184.0, 233: 182.4, 224: 181.9, 323: 170.7, 221: 174.0, 321: 171.3, 111: 299.6}),
    # one expert of 340 and of 300 rows: down
    (0, (16, 16, 0), 224, {741: 90.2, 751: 88.7, 641: 87.6, 831: 85.9, 531: 91.2, 111: 259.7}),
    (1, (16, 16, 0), 224, {741: 84.9, 751: 84.8, 641: 87.4, 831: 83.8, 531: 92.6, 111: 284.9}),
    (0, (16, 0, 16), 224, {813: 83.9, 814: 88.8, 713: 85.0, 714: 85.1, 812: 86.2, 815: 85.6, 111: 257.3}),
]


@pytest.mark.parametrize("fp8,tiles,kt,times", MEASURED)
def test_cut_is_near_the_best_measured(lib, fp8, tiles, kt, times):
    nsp = lib.ffn_cut(fp8, *tiles, NWG, kt, SPLIT_BYTES)
    digits = 100 * (nsp & 15) + 10 * (nsp >> 4 & 15) + (nsp >> 8)
    assert digits in times, (tiles, kt, digits)
    assert times[digits] <= 1.04 * min(times.values()), (tiles, kt, digits, times)
