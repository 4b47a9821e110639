"""The kernel of the 512 -> 128 -> 128 -> 512 bottleneck blocks with tiles of 32 and of 64 pixels, at their edges and in its three forms, against the oracle."""
import pytest

from test_gpu_block import run_block

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[1, 2], ids=["tiles32", "tiles64"])
def tile(request):
    from paper_2006_11735_amd import binding as B
    B.icnn_set_tuning("block128_tile", request.param)
    yield
    B.icnn_set_tuning("reset")


# one pixel, one row, one column (patches of as many rows as there are), whole tiles and ragged ones, more tiles than the chip holds at once
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 40), (1, 40, 1), (1, 4, 8), (1, 8, 8), (2, 13, 19), (3, 28, 28), (300, 5, 9)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("kw", [dict(), dict(skip=None), dict(forms=("hi", "wide")), dict(bound12=15)], ids=str)
def test_tiles(tile, shape, kw):
    got, want = run_block(sum(shape), *shape, 512, 128, **kw)
    assert (got == want).all(), "%d of %d bytes differ" % (int((got != want).sum()), want.size)
