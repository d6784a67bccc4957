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
import test_gpu_ffn_edges
import test_gpu_tile_families

SPLIT_BYTES = 128 * 256 * 256 * 4
NWG = 256


@pytest.fixture(scope="module")
def lib():
    so = ffn_host.load()
    so.ffn_cut.argtypes = [ctypes.c_int] * 6 + [ctypes.c_long]
    so.ffn_cut_cost.argtypes = [ctypes.c_int] * 6 + [ctypes.c_long, ctypes.c_int]
    so.ffn_cut_cost.restype = ctypes.c_double
    return so


def _check(lib, fp8, tiles, kt, nwg=NWG, split_bytes=SPLIT_BYTES):
    got = lib.ffn_cut(fp8, *tiles, nwg, kt, split_bytes)
    cuts = [a | b << 4 | c << 8 | h << 12 for a, b, c, h in itertools.product(*[range(1, 9)] * 3, range(2))]
    cost = {n: lib.ffn_cut_cost(fp8, *tiles, nwg, kt, split_bytes, n) for n in cuts}
    possible = {n: v for n, v in cost.items() if v >= 0}
    total = sum(tiles)
    if total % nwg == 0 or total // nwg >= 8:
        assert got == 0x111, (tiles, kt)
        return
    assert got in possible, (tiles, kt, hex(got))
    # times are compared in whole units of f32 sums
    assert possible[got] <= min(possible.values()) * (1 + 1e-5) + 1, (tiles, kt, hex(got))


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


# Measured times (us, weights in HBM) of launches under cuts worth having.  A
# cut is written as four digits: 2 where tiles are cut into column halves, then
# the pieces of the 256-, 128- and 64-row tiles.  The two weight formats, and
# launches of few and of many items, want different ones.
MEASURED = [
    # 8 experts of 111 .. 235 rows, d = 4096, f = 2048: gate/up, down
    (0, (96, 32, 0), 64, {2111: 71.2, 2121: 73.1, 2221: 83.4, 1221: 86.1, 1211: 89.7, 1111: 93.8}),
    (0, (96, 32, 0), 32, {2111: 41.7, 2121: 44.2, 1221: 49.2, 1211: 50.1, 1111: 55.8}),
    (1, (96, 32, 0), 32, {2111: 44.8, 2121: 45.2, 1211: 50.6, 1221: 50.7, 1111: 60.9}),
    # d = 4096, f = 14336, 400 tokens of 8 experts, top-2: down
    (0, (32, 32, 80), 224, {1233: 216.7, 1243: 220.2, 1223: 220.7, 1221: 229.6, 2321: 233.0, 2111: 259.8}),
    (1, (32, 32, 80), 224, {1321: 170.3, 1221: 173.2, 1332: 173.3, 1231: 176.2, 1322: 176.8, 2321: 190.9, 1323: 165.7}),
    # 777 tokens: down
    (0, (80, 48, 48), 224, {2111: 283.4, 1223: 284.6, 1222: 286.1, 1211: 297.1, 2222: 300.6, 1111: 313.4}),
    (1, (80, 48, 48), 224, {1222: 196.6, 1211: 206.3, 1212: 206.8, 2222: 246.6, 2111: 247.2}),
    # one expert of 340, 420, 800 and 60 rows: down, gate/up, down, gate/up
    (0, (16, 16, 0), 224, {2531: 79.0, 2431: 79.5, 2521: 80.9, 1641: 86.0, 1741: 86.5, 2111: 177.4, 1111: 259.5}),
    (1, (16, 16, 0), 224, {2531: 69.1, 2431: 74.0, 2441: 80.0, 1831: 83.6, 1741: 86.4, 2111: 189.4, 1111: 284.7}),
    (0, (224, 0, 0), 64, {1111: 94.9, 2111: 121.3}),
    (0, (48, 0, 16), 224, {1313: 118.7, 1312: 120.0, 1314: 122.2, 2211: 138.6, 2213: 152.7, 2111: 172.9}),
    (0, (0, 0, 112), 64, {2111: 49.5, 1112: 54.6, 2112: 60.4, 1111: 62.5}),
    # one expert of 174 rows, d = 3072, f = 1408: gate/up
    (0, (11, 0, 0), 48, {2411: 29.5, 2311: 30.4, 2511: 31.1, 1411: 39.7, 1511: 40.2, 2111: 46.0, 1111: 64.7}),
    # 22 experts of 16 rows, d = 4096, f = 2048: gate/up
    (0, (0, 0, 352), 64, {2111: 136.1, 1112: 139.4, 2112: 145.0, 2114: 146.2, 1111: 148.4}),
]


@pytest.mark.parametrize("fp8,tiles,kt,times", MEASURED)
def test_cut_is_near_the_best_measured(lib, fp8, tiles, kt, times):
    nsp = lib.ffn_cut(fp8, *tiles, NWG, kt, SPLIT_BYTES)
    digits = 1000 * (1 + (nsp >> 12)) + 100 * (nsp & 15) + 10 * (nsp >> 4 & 15) + (nsp >> 8 & 15)
    assert digits in times, (tiles, kt, digits)
    assert times[digits] <= 1.06 * min(times.values()), (tiles, kt, digits, times)


def _tiles(depths, cols):
    """Tiles per family of experts with these rows and this many column tiles."""
    n = [0, 0, 0]
    for r in depths:
        n[0] += r // 256 + (r % 256 > 128)
        n[1] += 64 < r % 256 <= 128
        n[2] += 0 < r % 256 <= 64
    return [v * cols for v in n]


def _launches(depths, d, f):
    """(tiles, K steps) of gate/up and down."""
    return (_tiles(depths, -(-f // 128)), d // 64), (_tiles(depths, -(-d // 256)), f // 64)


GPU_CASES = [(test_gpu_ffn_edges.CASES[n], c) for n, c in test_gpu_ffn_edges.CUTS.items()]
GPU_CASES += [(test_gpu_tile_families.SPLIT_CASES[n], c) for n, c in test_gpu_tile_families.CUTS.items()]


@pytest.mark.parametrize("fp8", [0, 1])
@pytest.mark.parametrize("case,cuts", GPU_CASES)
def test_gpu_cases_are_cut_as_they_say(lib, case, cuts, fp8):
    for (tiles, kt), cut in zip(_launches(*case), cuts):
        if cut is None:
            continue
        nsp = lib.ffn_cut(fp8, *tiles, NWG, kt, SPLIT_BYTES)
        assert sum(tiles) < NWG  # one partial round: every family is in the tail
        got = 1 + (nsp >> 12), tuple(f for f in range(3) if nsp >> (4 * f) & 15 > 1)
        assert got == cut, (tiles, kt, hex(nsp))
        if not cut[1]:
            assert all(tiles), tiles


@pytest.mark.parametrize("fp8", [0, 1])
def test_area_binds_in_its_gpu_case(lib, fp8):
    tiles, kt = _launches(*test_gpu_ffn_edges.CASES["area"])[1]
    assert lib.ffn_cut(fp8, *tiles, NWG, kt, SPLIT_BYTES) != lib.ffn_cut(fp8, *tiles, NWG, kt, 1 << 40)
