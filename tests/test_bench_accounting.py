"""What bench.py counts of the coupling matrix, against the rule of the launch counted out by hand."""
import numpy as np
import pytest

import bench


def by_hand(live, per):
    """Item by item: rows of tiles, slabs of `per` columns of tiles."""
    ct = live.shape[0]
    square, stored = 0, set()
    for row in range(ct):
        for first in range(0, ct, per):
            cols = range(first, min(first + per, ct))
            if 4 <= len(cols) <= 64 and not any(live[row, c] for c in cols):
                continue
            square += len(cols)
            stored |= {(max(row, c), min(row, c)) for c in cols}
    return square, len(stored)


# (tiles in a row, tiles of an item) of 64 .. 16384 representatives; 67 and 115 leave a last slab that is shorter, 67 one of two tiles
@pytest.mark.parametrize("ct,per", [(1, 1), (8, 1), (32, 2), (64, 4), (67, 5), (115, 8), (256, 32)])
@pytest.mark.parametrize("share", [0.0, 0.01, 0.2, 1.0])
def test_streamed_tiles(ct, per, share):
    rng = np.random.default_rng(ct)
    live = np.tril(rng.random((ct, ct)) < share, -1)
    live |= live.T
    assert bench.streamed_coupling_tiles(live) == by_hand(live, per)


def test_empty_and_short_items():
    none = np.zeros((256, 256), dtype=bool)
    assert bench.streamed_coupling_tiles(none) == (0, 0)
    one = none.copy()
    one[200, 3] = one[3, 200] = True                       # two items of 32 tiles, transposes of each other's neighbours
    assert bench.streamed_coupling_tiles(one) == (64, 63)
    assert bench.streamed_coupling_tiles(np.zeros((32, 32), dtype=bool)) == (1024, 528)      # items of two tiles: all of them


def test_tiles_with_a_value():
    torch = pytest.importorskip("torch")
    C = torch.zeros(130, 130)
    C[129, 1] = C[1, 129] = 0.5
    assert bench.live_coupling_tiles(torch, C, 3).tolist() == [[False, False, True], [False, False, False], [True, False, False]]
