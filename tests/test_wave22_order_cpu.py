"""The workgroup -> tile map of the 2 x 2 wave projection kernel (no GPU; not part of the C ABI, called by its C++ name): every
tile that holds rows once, column tiles on the XCD of their number, and no workgroup without work ahead of one with work in
an XCD's order, except that three row tiles are counted as four."""
import ctypes as C

import pytest

from paper_2602_06412_amd import binding as B


def _tile(wg, row_tiles, splits):
    out = (C.c_int * 3)()
    B.lib()._Z15slk_wave22_tileiiiPi(wg, row_tiles, splits, out)
    return tuple(out)


@pytest.mark.parametrize("launched,tiles_n,splits", [(2, 128, 1), (3, 128, 1), (4, 128, 1), (4, 115, 1), (2, 32, 4), (2, 21, 4), (2, 1, 1)])
@pytest.mark.parametrize("row_tiles", [1, 2, 3, 4])
def test_order(launched, tiles_n, splits, row_tiles):
    if row_tiles > launched:
        pytest.skip("no more row tiles than the launch has")
    grid = 8 * -(-tiles_n // 8) * (4 if launched == 3 else launched) * splits
    tiles = [_tile(wg, row_tiles, splits) for wg in range(grid)]
    working = [tm < row_tiles and tn < tiles_n for tm, tn, _ in tiles]
    got = [t for t, w in zip(tiles, working) if w]
    assert sorted(got) == [(tm, tn, s) for tm in range(row_tiles) for tn in range(tiles_n) for s in range(splits)]
    assert all(tn % 8 == wg % 8 for wg, (_, tn, _) in enumerate(tiles))
    for xcd in range(8):
        order = working[xcd::8]
        last = max(i for i, w in enumerate(order) if w) if any(order) else -1
        idle = [i for i, w in enumerate(order[:last + 1]) if not w]
        assert not idle or (row_tiles == 3 and all(i % 4 == 3 for i in idle))
