"""The order of the FFN kernels' LDS accesses, on the CPU.

The device code runs thread by thread on the host and every operand read and
direct-to-LDS load is recorded with the workgroup barriers and waits around
it.  Whatever a wave reads has to have landed before a barrier that precedes
the read, and has to be read completely before a barrier that precedes its
refill: no timing, however unlucky, may let a wave read bytes that another one
is replacing.  All waves must pass the same barriers."""

import ctypes

import pytest

import ffn_host


@pytest.fixture(scope="module")
def lib():
    so = ffn_host.load()
    so.ffn_order_violations.restype = ctypes.c_long
    return so


# whole rounds per family, tail (1: two pieces, 2: column halves, 3: both), this
# workgroup's arrival, XCD, two directions
CHAINS = {
    "family0": ((3, 0, 0), 0, 0, 0, 0),
    "family1": ((0, 3, 0), 0, 0, 0, 0),
    "family2": ((0, 0, 3), 0, 0, 0, 0),
    "families": ((2, 2, 2), 0, 0, 0, 0),
    "reversed": ((2, 2, 2), 0, 0, 1, 1),
    "pieces_first": ((1, 0, 0), 1, 0, 0, 0),
    "pieces_last": ((1, 0, 0), 1, 1, 0, 0),
    "pieces_reversed": ((1, 1, 1), 1, 1, 1, 1),
    "halves": ((0, 0, 0), 2, 0, 0, 0),
    "halves_last": ((1, 0, 0), 2, 0, 0, 0),
    "halves_reversed": ((1, 1, 1), 2, 0, 1, 1),
    "halves_pieces_first": ((1, 0, 0), 3, 0, 0, 0),
    "halves_pieces_last": ((0, 0, 0), 3, 1, 0, 0),
}


@pytest.mark.parametrize("fp8", [0, 1])
@pytest.mark.parametrize("gated", [0, 1])
@pytest.mark.parametrize("chain", sorted(CHAINS))
def test_lds_reads_and_refills_are_ordered(lib, chain, gated, fp8):
    whole, tail, arrival, xcd, mixed = CHAINS[chain]
    # fewer, as many and more K steps than a ring has stages, odd and even;
    # pieces need at least 8 steps each
    for kt in (16, 17, 23) if tail & 1 else (1, 2, 3, 4, 5, 13, 14):
        n, msg = ctypes.c_long(0), ctypes.create_string_buffer(256)
        bad = lib.ffn_order_violations(gated, fp8, kt, (ctypes.c_int * 3)(*whole), tail, arrival, xcd, mixed,
                                       ctypes.byref(n), msg, 256)
        assert n.value > 0 or bad
        assert bad != -1, f"{chain}, {kt} K steps: waves pass different numbers of barriers"
        assert bad == 0, f"{chain}, {kt} K steps: {bad} unordered accesses; {msg.value.decode()}"
