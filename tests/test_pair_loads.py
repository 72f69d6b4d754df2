"""Replay on the CPU of the loads and stores of neighbouring pairs.

The rows of shared 2D DoFs (neighbours2, edges.hpp), the restriction and the
prolongation (RestrictCell, ProlongCell, rows.hpp) access storage points two at
a time.  The second point of a pair, or the pair that stands in for a row the
point does not have, may lie outside the row: this replays the kernels' index
arithmetic for every point of every macro of small levels, and for edge slices
of the largest, and checks that both points of every pair lie in the macro's
storage, that neighbours inside the macro are taken from their storage index,
and that the prolongation writes every fine point exactly once.
"""
import numpy as np
import pytest

OFF2 = [(0, -1), (1, -1), (-1, 0), (0, 0), (1, 0), (-1, 1), (0, 1)]
OFF3 = [(0, 0, -1), (1, 0, -1), (0, 1, -1), (-1, 1, -1), (0, -1, 0), (1, -1, 0), (-1, 0, 0), (0, 0, 0),
        (1, 0, 0), (-1, 1, 0), (0, 1, 0), (0, -1, 1), (1, -1, 1), (-1, 0, 1), (0, 0, 1)]


def points(dim, N):
    return (N + 1) * (N + 2) // 2 * (1 if dim == 2 else N + 3) // (1 if dim == 2 else 3)


def row_start(S, y):
    return y * (S + 2) - (y * (y + 1)) // 2


def slice_base(N, z):
    t = lambda n: n * (n + 1) * (n + 2) // 6  # noqa: E731
    return t(N + 1) - t(N + 1 - z)


def index(dim, N, x, y, z):
    return row_start(N, y) + x if dim == 2 else slice_base(N, z) + row_start(N - z, y) + x


def slice_points(S):
    """x, y of a slice's points in storage order."""
    y = np.repeat(np.arange(S + 1), S + 1 - np.arange(S + 1))
    return np.arange(len(y)) - row_start(S, y), y


def inside(at, n, pair=True):
    return (at >= 0).all() and (at + (1 if pair else 0) < n).all()


@pytest.mark.parametrize("L", range(0, 9))
def test_neighbours_of_shared_points(L):
    N, P = 1 << L, points(2, 1 << L)
    x, y = slice_points(N)
    i = index(2, N, x, y, 0)
    x0, y0, far = x == 0, y == 0, x + y == N
    first, l = x0 & ~far, N + 1 - y
    at = np.where(first, 0, -1)
    m, s = i + at, i + np.where(y0, at, -l - 1)
    n = i + np.where(far, np.where(x0, at, l - 2), l - 1)
    e = i + np.where(far, 0, 1)
    assert inside(m, P) and inside(s, P) and inside(n, P) and inside(e, P, pair=False)
    got = [s, s + 1, m, np.where(first, m, m + 1), e, np.where(far, n + 1, n), n + 1]
    for g, (dx, dy) in zip(got, OFF2):
        k = (x + dx >= 0) & (y + dy >= 0) & (x + dx + y + dy <= N)
        assert np.array_equal(g[k], index(2, N, x + dx, y + dy, 0)[k]), (dx, dy)


def check_restriction(dim, Nc, z, anchor_off=0):
    """RestrictCell::load over the points of coarse slice z."""
    Nf, S = 2 * Nc, Nc - z
    x, y = slice_points(S)
    x0, y0, z0, far = x == 0, y == 0, dim == 2 or z == 0, x + y == S
    zf = 2 * z
    za = zf - 1 if dim == 3 and zf > 0 else 0
    Sf, yf = Nf - zf, 2 * y
    f = slice_base(Nf, za) if dim == 3 else 0
    tb = slice_base(Nf, zf) - slice_base(Nf, za) if dim == 3 else 0
    c, l = tb + row_start(Sf, yf) + 2 * x, Sf + 1 - yf
    P = points(dim, Nf) - f
    spare = np.maximum(c - 1, 0)
    pair = lambda ok, i: np.where(ok, i, spare)  # noqa: E731
    first = x0 & ~far
    D, xp = np.where(first, c, c - 1), np.where(far, c, c + 1)
    Cc, E = pair(~y0, c - l - 1), pair(~(far & x0), c + l - 1 + anchor_off)
    pairs = [D, Cc, E]
    v = [Cc, Cc + 1, D, np.where(first, D, D + 1), xp, E, E + 1]
    if dim == 3:
        dn, up = c - tb + yf, c + (Sf + 1) * (Sf + 2) // 2 - yf
        A, B = pair(not z0, dn), pair(not z0, dn + l)
        Ff, G = pair(~y0, up - l), pair(~(far & x0), up - 1)
        pairs += [A, B, Ff, G]
        v = [A, A + 1, B + 1, B] + v + [Ff, Ff + 1, G, G + 1]
    for p in pairs:
        assert inside(p, P) and (p * 8 < 2 ** 32).all()
    assert inside(xp, P, pair=False)
    for g, d in zip(v, OFF2 if dim == 2 else OFF3):
        fx, fy, fz = 2 * x + d[0], 2 * y + d[1], zf + (d[2] if dim == 3 else 0)
        k = (fx >= 0) & (fy >= 0) & (fz >= 0) & (fx + fy + fz <= Nf)
        if k.any():
            assert np.array_equal((f + g)[k], index(dim, Nf, fx[k], fy[k], fz)), d


def check_prolongation(dim, Nc, z, written=None):
    """ProlongCell over the points of coarse slice z; counts writes into `written`."""
    Nf, S = 2 * Nc, Nc - z
    X, Y = slice_points(S)
    room = S - X - Y
    Pc = points(dim, Nc)
    p = (slice_base(Nc, z) if dim == 3 else 0) + row_start(S, Y) + X
    l, up = S + 1 - Y, (S + 1) * (S + 2) // 2 - Y
    coarse = [(p + np.where(room >= 1, 1, 0), (1, 0, 0), room >= 1), (p + np.where(room >= 1, l, 0), (0, 1, 0), room >= 1)]
    if dim == 3:
        coarse += [(p + np.where(room >= 1, up, 0), (0, 0, 1), room >= 1),
                   (p + np.where(room >= 2, up + 1, 0), (1, 0, 1), room >= 2)]
    for at, d, k in coarse:
        assert inside(at, Pc, pair=False)
        if k.any():
            assert np.array_equal(at[k], index(dim, Nc, X[k] + d[0], Y[k] + d[1], z + d[2]))
    Sf, lf = 2 * S, 2 * S + 1 - 2 * Y
    uf = (Sf + 1) * (Sf + 2) // 2 - 2 * Y
    f = (slice_base(Nf, 2 * z) if dim == 3 else 0) + row_start(Sf, 2 * Y) + 2 * X
    at = [f, f + np.where(room >= 1, lf, 0)]
    if dim == 3:
        at += [f + np.where(room >= 1, uf, 0), f + np.where(room >= 1, uf + lf - 1, 0)]
    apex = (room == 0) & ((z if dim == 3 else Y) == Nc)
    NP = len(at)
    for k, a in enumerate(at):
        assert inside(a - apex, points(dim, Nf))
        py, pz = k & 1, k >> 1
        full = room >= 1
        if k == NP - 1 and dim == 3:
            full = room >= 2  # room = 1: the pair's first point alone
        for px in (0, 1):
            w = full if px or k else room >= 0
            if k == NP - 1 and dim == 3 and px == 0:
                w = room >= 1
            if w.any():
                to = index(dim, Nf, 2 * X[w] + px, 2 * Y[w] + py, 2 * z + pz)
                assert np.array_equal(a[w] + px, to), (k, px)
                if written is not None:
                    np.add.at(written, to, 1)


@pytest.mark.parametrize("L", range(0, 9))
def test_2d_transfers(L):
    Nc = 1 << L
    check_restriction(2, Nc, 0)
    w = np.zeros(points(2, 2 * Nc), dtype=np.int8)
    check_prolongation(2, Nc, 0, w)
    assert (w == 1).all()


@pytest.mark.parametrize("L", range(0, 6))
def test_3d_transfers(L):
    Nc = 1 << L
    w = np.zeros(points(3, 2 * Nc), dtype=np.int8)
    for z in range(Nc + 1):
        check_restriction(3, Nc, z)
        check_prolongation(3, Nc, z, w)
    assert (w == 1).all()


@pytest.mark.parametrize("z", [0, 1, 2, 511, 1022, 1023, 1024])
def test_3d_transfers_into_level_11(z):
    check_restriction(3, 1 << 10, z)
    check_prolongation(3, 1 << 10, z)


def test_replay_catches_a_pair_past_the_macro():
    with pytest.raises(AssertionError):
        check_restriction(2, 4, 0, anchor_off=1)
