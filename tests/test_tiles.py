"""Tiles of the run-time-length passes against the limits of a launch, on the host: the dynamic LDS of
every tile that the library may choose fits a workgroup beside what the kernels declare themselves."""
import ctypes

import pytest

LDS_PER_WORKGROUP = 160 * 1024
STATIC = 64  # the block sum of a pass kernel: one double per wavefront, at most 8
MAX_THREADS, MAX_PRODUCTS = 512, 4


class Axis(ctypes.Structure):
    _fields_ = [("L", ctypes.c_int), ("nst", ctypes.c_int), ("rad", ctypes.c_int * 16), ("q", ctypes.c_int),
                ("p", ctypes.c_int), ("tw", ctypes.c_int)]


class Tile(ctypes.Structure):
    _fields_ = [("ok", ctypes.c_bool), ("n", ctypes.c_int), ("threads", ctypes.c_int), ("ni", ctypes.c_int),
                ("lds", ctypes.c_size_t)]


def axis(L):
    """A length's split into q p: two register radices (up to 17) as equal as possible, else the largest
    register radix and a dense step; the larger one first in the middle pass's register form (<= 9)."""
    q, p = 1, L
    for r in range(1, 18, 2):
        if L % r:
            continue
        if L // r <= 17 and r > L // r:
            break
        q, p = r, L // r
    return Axis(L=L, q=p, p=q) if p <= 9 else Axis(L=L, q=q, p=p)


@pytest.fixture(scope="module")
def tiles():
    from paper_1508_02045_amd import fgh
    L = fgh.lib()
    row, ax, mid = (getattr(L, n) for n in ("_ZN3fgh12gen_row_tileERKNS_4AxisEixmi",
                                            "_ZN3fgh13gen_axis_tileERKNS_4AxisEixm",
                                            "_ZN3fgh12gen_mid_tileERKNS_4AxisEim"))
    for f, args in ((row, [ctypes.c_int, ctypes.c_longlong, ctypes.c_size_t, ctypes.c_int]),
                    (ax, [ctypes.c_int, ctypes.c_longlong, ctypes.c_size_t]),
                    (mid, [ctypes.c_int, ctypes.c_size_t])):
        f.restype = Tile
        f.argtypes = [ctypes.POINTER(Axis)] + args
    return row, ax, mid


def check(t, what):
    if not t.ok:
        return 0
    assert t.lds + STATIC <= LDS_PER_WORKGROUP, (what, t.n, t.lds)
    assert t.n >= 1 and 64 <= t.threads <= MAX_THREADS and t.threads % 64 == 0 and 0 <= t.ni <= MAX_PRODUCTS, what
    return 1


EXTENTS = [3, 5, 9, 21, 45, 99, 151, 243, 511, 513, 999, 1941, 2659, 4095, 8191, 65535, 1 << 20]


@pytest.mark.parametrize("cs", [8, 16])
def test_every_tile_can_be_launched(tiles, cs):
    row, ax, mid = tiles
    n = 0
    for L in range(3, 8192, 2):
        a = axis(L)
        for x in EXTENTS:
            for d in (2, 3):
                n += check(row(a, d, x, cs, 32), ("row", L, d, x, cs))
            n += check(mid(a, x, cs), ("middle", L, x, cs))
            for inner in (2, 8, 51, 122):
                n += check(ax(a, inner, 3 * x, cs), ("axis", L, inner, x, cs))
    assert n > 100000


def test_known_full_tiles(tiles):
    """Lengths whose best tile is only just too large: a smaller one is taken, not refused."""
    row, ax, mid = tiles
    for L, d, rows in ((3381, 2, 3), (1449, 3, 2025)):
        t = row(axis(L), d, rows, 16, 32)
        assert check(t, ("row", L, d, rows)), (L, d, rows)
