"""How many query rows a workgroup of the attention gets (a host function of sizes): by the time a launch of either height takes,
given where its rows lie."""
import heapq
import random

from paper_2505_07203_amd import binding as B

UNITS, ENDS, SHARE = 256, 5, 0.6      # compute units; key tiles for a workgroup's ends; a key tile of 128 rows in ones of 256


def span(N, q_row0, Hq, rows):
    """key tiles until the last workgroup ends: longest first, each to the unit that is free first"""
    free = [0] * UNITS
    for tile in range((N - 1) // rows, q_row0 // rows - 1, -1):
        keys = (min(N, (tile + 1) * rows) - 1) // 64 + 1 + ENDS
        for _ in range(Hq):
            heapq.heapreplace(free, free[0] + keys)
    return max(free)


def test_rows_by_expected_time():
    rng = random.Random(3)
    heights = {128: 0, 256: 0}
    for i in range(400):
        Hq = rng.choice([1, 8, 20, 32, 40, 64, 128, 256])
        n = rng.randint(1, 256 * 256 // Hq)
        q0 = rng.choice([0, rng.randint(1, 20000)])
        rows = B.po_attention_tile(q0 + n, Hq, Hq, 128, q0)
        heights[rows] += 1
        t128, t256 = SHARE * span(q0 + n, q0, Hq, 128), span(q0 + n, q0, Hq, 256)
        one_round = (-(-(q0 + n) // 256) - q0 // 256) * Hq <= UNITS
        if rows == 128:
            assert one_round and t128 < t256 * 1.001, (Hq, n, q0)
        else:       # (a unit that is free early may take two short workgroups in the simulation)
            assert not one_round or t128 > t256 * 0.97, (Hq, n, q0)
    assert min(heights.values()) > 50


def test_causal_launches_of_one_round_and_suffixes():
    for Hq, Hkv, top in ((32, 8, 2048), (40, 8, 1536), (20, 4, 3072)):
        assert {B.po_attention_tile(n, Hq, Hkv) for n in range(1, top + 1)} == {128}
        assert B.po_attention_tile(top + 1, Hq, Hkv) == 256
    # behind a cached prefix all tiles are about as long: 128 rows until they take a second round
    for n, rows in ((1, 128), (150, 128), (900, 128), (1000, 256), (1100, 256), (1800, 256), (1900, 256)):
        assert B.po_attention_tile(14000 + n, 32, 8, 128, 14000) == rows, n
    # plain queries, the other head dimension
    assert B.po_attention_tile(100, 32, 8, 128, 0, False) == B.po_attention_tile(100, 32, 8, 64) == 256


def test_launches_of_the_gpu_tests_start_inside_tiles_of_both_heights():
    """suffixes behind a cached prefix and the last layer's single row, as in test_gpu_out_of_range.py"""
    at = {(B.po_attention_tile(n, 32, 8, 128, q0), q0 % 128 != 0) for n in (2000, 2300, 4500)
          for q0 in (0, 1000, n - 1100, n - 300, n - 70, n - 1)}
    assert at >= {(128, True), (256, True), (256, False)}


def test_arguments():
    L, r = B.lib(), B.C.c_int32(0)
    ask = lambda *a: L.po_attention_tile(*a, B.C.byref(r))
    assert ask(0, 4, 2, 128, 0, 1) == ask(9, 4, 3, 128, 0, 1) == ask(9, 4, 2, 128, 9, 1) == B.PO_ERR_INVALID_ARG
    assert L.po_attention_tile(9, 4, 2, 128, 0, 1, None) == B.PO_ERR_INVALID_ARG
    assert ask(9, 4, 2, 96, 0, 1) == B.PO_ERR_BAD_CONFIG
