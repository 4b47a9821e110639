"""The kernel of the 256 -> 64 -> 64 -> 256 bottleneck blocks (iconv2d_bottleneck_brelu) at the edges of its tiles, against the oracle."""
import pytest

from test_gpu_block import run_block

pytestmark = pytest.mark.gpu


# one tile, one pixel, tiles ragged on both axes, one row, one column, more tiles than the chip holds at once
@pytest.mark.parametrize("shape", [(1, 4, 14), (1, 1, 1), (2, 13, 19), (1, 1, 70), (1, 70, 1), (3, 28, 28), (210, 12, 12)], ids=lambda s: "x".join(map(str, s)))
def test_tiles(shape):
    got, want = run_block(sum(shape), *shape, 256, 64)
    assert (got == want).all(), "%d of %d bytes differ" % (int((got != want).sum()), want.size)


def test_a_picture_taller_than_16384_rows():
    # tiles of 8 x 7 = 56 of 64 pixel slots: the other eight belong to nobody, at any height
    got, want = run_block(3, 1, 16500, 7, 256, 64)
    assert (got == want).all(), "%d of %d bytes differ" % (int((got != want).sum()), want.size)


# tiles of 4 x 14: first and last pixel 253 apart, 2 GiB at 8.49 million channels from pixel to pixel; on either side of it
@pytest.mark.parametrize("pitch", [8488064, 8488080, 9437184])
def test_a_tile_over_two_gib_of_output(pitch):
    got, want = run_block(4, 1, 4, 80, 256, 64, pitch=pitch)
    assert (got == want).all(), "%d of %d bytes differ" % (int((got != want).sum()), want.size)


@pytest.mark.parametrize("kw", [dict(skip=None), dict(skip="s32"), dict(c3_mode="linear_s8", skip=None), dict(c3_mode="raw_s32"), dict(forms=("hi", "hi")),
                                dict(forms=("wide", "hi")), dict(bound12=15), dict(cbuf=320)], ids=str)
def test_output_and_skip_modes(kw):
    # (int32 operands and outputs, inputs of another pitch than the skip operand's, and shifts beyond 32 stay on the other kernels)
    got, want = run_block(7, 2, 11, 13, 256, 64, **kw)
    assert (got == want).all()


def test_the_other_kernel_gives_the_same_bytes():
    from paper_2006_11735_amd import binding as B
    got, want = run_block(5, 2, 56, 56, 256, 64)
    B.icnn_set_tuning("no_block64s", 1)
    try:
        other, _ = run_block(5, 2, 56, 56, 256, 64)
    finally:
        B.icnn_set_tuning("reset")
    assert (got == want).all() and (got == other).all()
