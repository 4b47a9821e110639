"""The kernel of small workgroups on the 64 -> 64 -> 64 -> 256 blocks with a projection (iconv2d_bottleneck_dual_brelu) at the edges of its tiles and of
the rescale it takes (shifts below 32), against the oracle."""
import pytest

from test_gpu_block import run_proj_block

pytestmark = pytest.mark.gpu


# one tile, one pixel, tiles ragged on both axes, one row, one column, taller than 16384 rows, more tiles than the chip holds at once
@pytest.mark.parametrize("shape", [(1, 4, 14), (1, 1, 1), (2, 13, 19), (1, 1, 70), (1, 70, 1), (1, 16500, 7), (3, 28, 28), (210, 12, 12)],
                         ids=lambda s: "x".join(map(str, s)))
def test_tiles(shape):
    got, want = run_proj_block(sum(shape), *shape)
    assert (got == want).all(), "%d of %d bytes differ" % (int((got != want).sum()), want.size)


@pytest.mark.parametrize("pair", [(2, 0), (3, 1), (1 << 30, 31), (3 << 29, 32), (3 << 29, 34)], ids=str)
@pytest.mark.parametrize("c3_mode", ["brelu", "linear_s8"])
def test_rescale(pair, c3_mode):
    got, want = run_proj_block(11, 2, 11, 13, cbuf=80, c3_mode=c3_mode, res_pair=pair)
    assert (got == want).all(), "%d of %d bytes differ" % (int((got != want).sum()), want.size)


def test_the_other_kernel_gives_the_same_bytes():
    from paper_2006_11735_amd import binding as B
    got, want = run_proj_block(5, 2, 56, 56)
    B.icnn_set_tuning("no_block64s", 1)
    try:
        other, _ = run_proj_block(5, 2, 56, 56)
    finally:
        B.icnn_set_tuning("reset")
    assert (got == want).all() and (got == other).all()
