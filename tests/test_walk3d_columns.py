"""Replay on the CPU of the 3D walk's column decode and offsets (walk3d.hpp).

A slab's columns are numbered band by band (band b of side A has A - R b);
every lane finds its band from its number with an FP32 root that may be an ulp
off, and its rows' storage offsets by additions.  The decode must be exact at
every column, and the offsets of the rows a written point reads must be the
layout's, up to the largest level.
"""
import numpy as np
import pytest

F = np.float32


def band_starts(A, R):
    b = np.arange((A - 2) // R + 2, dtype=np.int64)
    return b * A - R * ((b * (b - 1)) >> 1)


def columns(A, R, q, ulp):
    c = F(2 * A + R)
    root = np.sqrt(np.maximum(c * c - F(8 * R) * q.astype(F), F(0))).astype(F)
    if ulp:
        root = np.nextafter(root, F(np.inf * ulp)).astype(F)
    b = np.maximum(((c - root) * F(0.5 / R)).astype(np.int64), 0)
    start = lambda k: k * A - R * ((k * (k - 1)) >> 1)  # noqa: E731
    lo = start(b) > q
    hi = ~lo & (start(b + 1) <= q)
    b = b - lo + hi
    return q - start(b), R * b


@pytest.mark.parametrize("R", [1, 2, 3, 4])
def test_every_column_decodes(R):
    for A in list(range(2, 260)) + [511, 1023, 1024, 1500, 2040, 2047]:
        s = band_starts(A, R)
        lens = np.array([A - R * b for b in range(len(s)) if A - R * b >= 2])
        Q = int(lens.sum())
        q = np.arange(Q, dtype=np.int64)
        b = np.repeat(np.arange(len(lens)), lens)
        for ulp in (0, -1, 1):
            x, y0 = columns(A, R, q, ulp)
            assert np.array_equal(y0, R * b) and np.array_equal(x, q - s[b]), (A, R, ulp)


def row_start(S, y):
    return y * (S + 2) - ((y * (y + 1)) >> 1)


def slice_base(N, z):
    t = lambda n: n * (n + 1) * (n + 2) // 6  # noqa: E731
    return t(N + 1) - t(N + 1 - z)


@pytest.mark.parametrize("N,R,PZ,E", [(16, 1, 2, 8), (64, 2, 4, 4), (128, 3, 4, 8), (256, 4, 6, 8), (2048, 4, 8, 8)])
def test_offsets_are_the_layouts(N, R, PZ, E):
    """Offsets of rows y0 .. y0 + R + 1 of slices z0 - 1 .. z0 + PZ, advanced as the kernel advances them, for the
    columns at both ends of the first, a middle and the last bands."""
    for z0 in [z for z in (1, 1 + PZ, (N // 2 - 1) // PZ * PZ + 1, (N - 3) // PZ * PZ + 1) if z <= N - 2]:
        A = N - z0
        nz = min(PZ, N - 1 - z0)
        nb = (A - 2) // R + 1
        rest = (slice_base(N, N + 1) - slice_base(N, z0 - 1)) * E
        for b in sorted({0, 1, nb // 2, nb - 1} & set(range(nb))):
            for x in sorted({0, 1, A - R * b - 1}):
                y0 = R * b
                o, D, S = (row_start(A + 1, y0) + x) * E, (A + 2 - y0) * E, A + 1
                for i in range(nz + 2):
                    r, z = o, z0 - 1 + i
                    for j in range(R + 2):
                        if x + y0 + j + z <= N:
                            assert r == (slice_base(N, z) - slice_base(N, z0 - 1) + row_start(N - z, y0 + j) + x) * E
                            assert r + E <= rest
                        assert 0 <= r < 2 ** 31
                        r += D - j * E
                    o += (((S + 1) * (S + 2)) >> 1) * E - y0 * E
                    D -= E
                    S -= 1
