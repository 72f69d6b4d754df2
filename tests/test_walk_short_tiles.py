"""Replay on the CPU of the 2D walk's loads for the tiles of two and four rows, and
of the condition under which a tile takes the unclamped path.

Tiles of levels that need few of them are two or four rows high with a load ring
as deep; their loads are replayed as those of the taller ones are (lane by lane,
against the macro's storage).  The pass that makes the first two sweeps at once
scales every value it reads by the interior's diagonal on the unclamped path, so
no row that such a tile reads may hold a point of the macro's boundary.
"""
import pytest

from test_walk_addresses import LANES, W62, check_2d, inner2d, loads_tile2d_fast, rs32, tiles2d

SHORT = [(2, 2), (4, 4)]


def inner_two_sweeps(x0, y0, N, H):
    return x0 >= 2 and y0 >= 2 and x0 + y0 + W62 + H + 1 <= N


@pytest.mark.parametrize("L", range(0, 9))
@pytest.mark.parametrize("H,U", SHORT)
def test_every_tile(L, H, U):
    N = 1 << L
    assert check_2d(N, H, U, tiles2d(N, H)) > 0
    assert check_2d(N, H, U, tiles2d(N, H), with_b=False) > 0


@pytest.mark.parametrize("H", [2, 4, 8, 16])
@pytest.mark.parametrize("L", [8, 9])  # (level 7 has no such tile)
def test_two_sweeps_read_no_boundary_point_unclamped(L, H):
    N = 1 << L
    taken = 0
    for x0, y0 in tiles2d(N, H):
        if not inner_two_sweeps(x0, y0, N, H):
            continue
        assert inner2d(x0, y0, N, H)
        taken += 1
        for r, off in loads_tile2d_fast(x0, y0, N, H):
            x = off - rs32(N, r)
            assert r >= 1 and (x == x0 - 1 + LANES).all() and x.min() >= 1 and x.max() + r < N, (x0, y0, r)
    assert taken > 0


def test_replay_catches_the_margin_of_one_sweep():
    """Without the extra margin a tile's first column of reads would be x = 0."""
    x0, y0, N, H = 1, 2, 256, 8
    assert inner2d(x0, y0, N, H) and not inner_two_sweeps(x0, y0, N, H)
    assert min(int((off - rs32(N, r)).min()) for r, off in loads_tile2d_fast(x0, y0, N, H)) == 0
