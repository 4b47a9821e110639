"""The kernel of the blocks of 64 middle channels and 256 outer ones in tiles of 32 and of 64 pixels, at the edges of either and of the choice between them, against the
oracle."""
import pytest

from test_gpu_block import run_block, run_proj_block

pytestmark = pytest.mark.gpu


# one pixel, a tile that is full (4 x 7, 4 x 14), ragged on both axes, a row, a column, several tiles to a workgroup, 256 tiles of 32 pixels and
# one more picture, 300 tiles of 64 pixels (600 of 32: the small ones) and 400 (800 of 32: the large ones)
@pytest.mark.parametrize("tile", [1, 2, 0])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 4, 7), (1, 4, 14), (2, 13, 19), (1, 1, 70), (1, 70, 1), (330, 8, 14), (64, 8, 14), (65, 8, 14), (150, 8, 14), (200, 8, 14)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("block", ["identity", "opening"])
def test_tiles(block, shape, tile):
    from paper_2006_11735_amd import binding as B
    B.icnn_set_tuning("block64s_tile", tile)
    try:
        got, want = run_block(sum(shape), *shape, 256, 64) if block == "identity" else run_proj_block(sum(shape), *shape)
    finally:
        B.icnn_set_tuning("reset")
    assert (got == want).all(), "%d of %d bytes differ" % (int((got != want).sum()), want.size)


@pytest.mark.parametrize("kw", [dict(skip=None), dict(c3_mode="linear_s8", skip=None), dict(bound12=15)], ids=str)
def test_output_and_skip_modes_in_small_tiles(kw):
    got, want = run_block(7, 2, 11, 13, 256, 64, **kw)
    assert (got == want).all()
