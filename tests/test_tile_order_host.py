"""The order in which query tiles are handed to the kernels, against its definition tile by tile."""
import random

import numpy as np
import pytest

import paper_2503_07680_amd as H


def key_tiles(tile, cu):
    n_keys = tile[3] - int(cu[tile[0]])          # of the tile's last row
    return -(-n_keys // 64)


@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("lengths", [[1], [64], [65, 64, 63], [129, 128, 300], [1] * 700, [256] * 600,
                                     [641] + [3] * 511, [4096, 130, 4097, 8191]])
def test_most_key_tiles_first_and_the_plans_order_among_equals(lengths, rows):
    cu, _, tiles, _, _ = H.hbp_pack_plan(lengths, sum(lengths), rows, H.HBP_TILES_QUERY)
    got = H.hbp_order_query_tiles(cu, tiles)
    plan = [tuple(t) for t in tiles.tolist()]
    want = sorted(plan, key=lambda t: -key_tiles(t, cu))          # stable
    assert got.dtype == np.int32 and got.flags["C_CONTIGUOUS"] and [tuple(t) for t in got.tolist()] == want
    assert [tuple(t) for t in tiles.tolist()] == plan             # the plan itself stays as it is


def test_a_tail_of_one_row_goes_with_its_full_neighbour():
    rnd = random.Random(5)
    lengths = [rnd.randint(16, 600) for _ in range(40)] + [1025]
    cu, _, tiles, _, _ = H.hbp_pack_plan(lengths, sum(lengths), 128, H.HBP_TILES_QUERY)
    order = [tuple(t) for t in H.hbp_order_query_tiles(cu, tiles).tolist()]
    assert [t[3] - t[2] for t in order[:2]] == [1, 128] and order[0][0] == order[1][0] == 40


def test_an_empty_plan():
    cu, _, tiles, _, _ = H.hbp_pack_plan([], 16, 128, H.HBP_TILES_QUERY)
    assert H.hbp_order_query_tiles(cu, tiles).shape == (0, 4)


def test_what_is_no_tile_of_the_pack_is_refused():
    cu, _, tiles, _, _ = H.hbp_pack_plan([200, 130], 330, 128, H.HBP_TILES_QUERY)
    for column, value in ((0, 2), (0, -1), (3, 0), (3, 331)):
        bad = tiles.copy()
        bad[1, column] = value
        with pytest.raises(H.HbpError) as e:
            H.hbp_order_query_tiles(cu, bad)
        assert e.value.status == 1
    lib = H.load_library()
    out = tiles.copy()
    at, cu_at, to = tiles.ctypes.data, cu.ctypes.data, out.ctypes.data
    for args in ((None, 2, at, 4, to), (cu_at, 2, None, 4, to), (cu_at, 2, at, 4, None), (cu_at, 2, at, -1, to),
                 (cu_at, -1, at, 4, to)):
        assert lib.hbp_order_query_tiles(*args) == 1
    assert lib.hbp_order_query_tiles(None, 0, None, 0, None) == 0 and np.array_equal(out, tiles)
