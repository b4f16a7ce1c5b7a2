"""The choice of the rounds launch's tiles (csrc/rounds.hip), on the host: the
smallest tiles for the frame's size of which it has at most 2.5 per compute
unit (256 units), larger ones where that takes them, and the smaller ones again
where none of the table does."""
import ctypes
import math

import pytest

TILES = {1: (32, 8), 2: (32, 16), 3: (32, 32), 4: (64, 16), 5: (64, 32), 6: (64, 8), 7: (64, 16)}
PIXELS = {1: 1, 2: 1, 3: 1, 4: 4, 5: 4, 6: 2, 7: 2}  # per thread and row


@pytest.fixture(scope="module")
def abi():
    from paper_1509_04232_amd import _abi
    _abi.lib.slic_test_rounds_variant.argtypes = [ctypes.c_void_p, ctypes.c_int32]
    return _abi


def _choice(abi, w, h, S, n=10):
    p = abi.SlicParams(w, h, 3 * w, 3, S, 0, 10.0, 0, 0)
    return abi.lib.slic_test_rounds_variant(ctypes.byref(p), n)


def _tiles(w, h, S, v):
    """Tiles of variant v, or None where the launch does not take them."""
    if S > 85 or S % PIXELS[v] or w % PIXELS[v]:
        return None
    (tw, th) = TILES[v]
    tx, ty = -(-w // tw), -(-h // th)

    def most(tile, step, n):
        return (tile - math.gcd(tile, step) + n - 1) // tile + 1

    cells = [(S - math.gcd(t, S) + t - 1) // S + 3 for t in (tw, th)]
    sources = min(most(tw, S, 3 * S), tx) * min(most(th, S, 3 * S), ty)
    window = cells[0] * cells[1]
    words = 34 * 16 + 2 * tx * ty + 2 * tx * ty * window * 4
    if tx * ty > 1024 or sources > 16 or window > 64 or words * 8 > 8 * w * h:
        return None
    return tx * ty


@pytest.mark.parametrize("w,h,S,want", [
    (320, 240, 16, 1), (640, 480, 16, 2), (720, 576, 16, 3), (800, 600, 20, 3), (1000, 700, 20, 5),
    (1024, 1024, 32, 5), (1280, 720, 16, 5), (1920, 1080, 8, 5), (933, 800, 27, 3),
    # no 32 x 8 tiles (a cell meets more than sixteen): 32 x 16, not more
    (144, 78, 32, 2), (82, 121, 20, 2),
    (3631, 3859, 84, 0), (64, 48, 86, 0),
])
def test_tiles_of_known_frames(abi, w, h, S, want):
    assert _choice(abi, w, h, S) == want


@pytest.mark.parametrize("S", [2, 4, 7, 8, 10, 13, 16, 20, 27, 32, 48, 64, 85])
def test_tiles_follow_the_rule(abi, S):
    for w, h in [(33, 40), (96, 72), (144, 78), (200, 150), (320, 240), (333, 251), (512, 256),
                 (640, 480), (654, 512), (720, 576), (801, 601), (1030, 700), (1280, 720), (1366, 768),
                 (1600, 900), (1920, 1080), (1921, 1080), (2400, 1400)]:
        px = w * h
        least = 1 if px <= 1 << 17 else 2 if px <= 1 << 19 else None
        got = _choice(abi, w, h, S)
        if got == 0:
            for v in (least, 2) if least else (3, 4, 5):
                if v and (n := _tiles(w, h, S, v)) is not None:
                    # only a variant that the association would not take there
                    assert least is None and n > 640, (w, h, S, v)
            continue
        n = _tiles(w, h, S, got)
        assert n is not None, (w, h, S, got)
        smaller = [v for v in range(least or 3, got) if v <= 3] if n <= 640 else []
        for v in smaller:  # those before it in the order have too many tiles
            m = _tiles(w, h, S, v)
            assert m is None or m > 640, (w, h, S, got, v)
        if n > 640:
            assert all((m := _tiles(w, h, S, v)) is None or m > 640 for v in (least or 3, 3, 5))


def test_one_round_and_too_many_have_no_such_launch(abi):
    assert _choice(abi, 640, 480, 16, 1) == 0
    assert _choice(abi, 640, 480, 16, 16384) == 0
    assert _choice(abi, 640, 480, 16, 16383) == 2
