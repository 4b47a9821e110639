"""The 3x3 kernel of 64 -> 64 channels that keeps its weights in registers, at the edges of its rounds, tiles and pictures and in the forms it takes, against
the oracle; calls that it leaves to the others; and the library's choice."""
import numpy as np
import pytest

from oracle import oracle as O
from test_gpu_flat import check, layer

pytestmark = pytest.mark.gpu


@pytest.fixture
def keep():
    from paper_2006_11735_amd import binding as B
    B.icnn_set_tuning("keep", 1)
    yield
    B.icnn_set_tuning("reset")


def skip_of(g, n, h, w):
    return dict(res=g.integers(0, 128, size=(n, h, w, 64), dtype=np.uint8), res_mode="pre", res_mul=20000, res_shift=5)


# one pixel, rounds of 128 pixels less and more one, a row, a column, many small pictures, rows of all widths up to the widest it takes, one and two rounds a
# workgroup and some with one more than the others
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 126), (1, 127, 1), (1, 16, 8), (1, 43, 3), (300, 2, 3), (130, 1, 1), (5, 7, 7), (3, 14, 14), (2, 28, 28), (1, 56, 56),
                                   (3, 9, 126), (2, 31, 57), (1, 112, 112), (11, 56, 56), (700, 7, 7), (90, 28, 29)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("skip", [False, True], ids=["plain", "skip"])
def test_tiles(keep, shape, skip):
    g, x, wt, b = layer(sum(shape), *shape, 64, 64, 3)
    check(x, wt, b, mul=32767, shift=25, **(skip_of(g, *shape) if skip else {}))


def tiles_of(n, h, w):
    """The workgroups' tiles, in rounds, as the launch deals them out"""
    def buffer(rounds):
        rows, pitch = (128 * rounds + w - 2) // w + 1, ((w + 2) * 80 + 1023) // 1024 * 1024
        return max((rows + 2 + (rows + h - 2) // h) * pitch, 36 * 1024)
    rounds = (n * h * w + 127) // 128
    workgroups = 8 * min(32, (rounds + 7) // 8)
    longest, most = -(-rounds // workgroups), 1
    while most < 8 and 2 * buffer(most + 1) <= 160 * 1024:
        most += 1
    start = min(2, most)
    rest = max(longest - start, 1)
    most = max(-(-rest // -(-rest // most)), start)
    found = set()
    for mine in {rounds // workgroups, longest}:
        tiles = [min(start, mine)]
        while sum(tiles) < mine:
            tiles.append(min(most, mine - sum(tiles)))
        found.add(tuple(tiles))
    return found


# tiles that follow one another: two and more, so that a buffer is used again, of one to four rounds each, of odd and even numbers of them, whole pictures and parts
@pytest.mark.parametrize("shape, tiles", [((97, 32, 32), {(2, 1), (2, 2)}), ((700, 1, 126), {(1, 1), (1, 1, 1)}), ((700, 14, 14), {(2, 2), (2, 3)}),
                                          ((900, 14, 14), {(2, 2, 1), (2, 2, 2)}), ((16, 112, 112), {(2, 3, 1), (2, 3, 2)}), ((1500, 14, 14), {(2, 3, 3), (2, 3, 3, 1)}),
                                          ((128, 56, 56), {(2, 4, 4, 2), (2, 4, 4, 3)})], ids=str)
@pytest.mark.parametrize("skip", [False, True], ids=["plain", "skip"])
def test_several_tiles(keep, shape, tiles, skip):
    assert tiles_of(*shape) == tiles
    g, x, wt, b = layer(sum(shape), *shape, 64, 64, 3)
    check(x, wt, b, mul=32767, shift=25, **(skip_of(g, *shape) if skip else {}))


@pytest.mark.parametrize("kw", [dict(), dict(out_mode="linear_s8"), dict(out_mode="clamp_u8", lo=3, hi=250), dict(bound_q=15), dict(mul=20001, shift=24), dict(mul=1, shift=9)], ids=str)
@pytest.mark.parametrize("skip", [False, True], ids=["plain", "skip"])
@pytest.mark.parametrize("inputs", ["unsigned", "signed", "pitch"])
def test_forms(keep, kw, skip, inputs):
    g, x, wt, b = layer(7, 2, 19, 23, 64, 64, 3, pitch=32 if inputs == "pitch" else 0, signed=inputs == "signed")
    check(x, wt, b, **kw, **(skip_of(g, 2, 19, 23) if skip else {}))


# what it does not take goes where it went before: too wide a picture, int32 sums, other operands, a wide multiplier, parameters per channel, inputs up to 255
@pytest.mark.parametrize("how", ["wide", "raw", "s8", "post", "multiplier", "channels", "255"])
def test_left_to_the_others(keep, how):
    from test_gpu_conv import channel_params
    n, h, w = (1, 5, 127) if how == "wide" else (2, 11, 13)
    g, x, wt, b = layer(3, n, h, w, 64, 64, 3)
    if how == "255":
        x = 2 * x + 1
    more = {"wide": {}, "255": {}, "raw": dict(out_mode="raw_s32"), "multiplier": dict(mul=2**31 - 1, shift=43), "channels": channel_params(3, 64),
            "s8": dict(res=g.integers(-128, 128, size=(n, h, w, 64)).astype(np.int8), res_mode="pre", res_mul=20000, res_shift=5),
            "post": dict(res=g.integers(0, 128, size=(n, h, w, 64), dtype=np.uint8), res_mode="post", res_mul=20000, res_shift=15)}[how]
    check(x, wt, b, **more)


# the library's choice on both sides of its lines: one round of another kernel's workgroups, and beyond
@pytest.mark.parametrize("shape", [(44, 32, 32), (45, 32, 32), (96, 32, 32), (97, 32, 32), (1, 400, 246), (1, 262, 263)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("skip", [False, True], ids=["plain", "skip"])
def test_the_librarys_choice(shape, skip):
    from gpu_util import gpu_conv2d
    from paper_2006_11735_amd import binding as B
    g, x, wt, b = layer(2, *shape, 64, 64, 3)
    kw = dict(pad=1, mul=20000, shift=25, **(skip_of(g, *shape) if skip else {}))
    got = gpu_conv2d(x, wt, b, **kw)
    B.icnn_set_tuning("tile", 1)                       # the tap-by-tap kernel
    try:
        want = gpu_conv2d(x, wt, b, **kw)
    finally:
        B.icnn_set_tuning("reset")
    assert got.max() > got.min() and (got == want).all()
