"""GPU parity of chains whose waves have none, one or several pixel groups of a layer (the last one takes the next layer's weights), in both
requantisation forms, against the oracle, bit for bit."""
import pytest

from test_gpu_chain import run_chain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(1, 1), (3, 5), (4, 9), (1, 40), (12, 12), (16, 16), (19, 22)], ids=str)
@pytest.mark.parametrize("layers", [2, 3, 6])
def test_pixel_groups_of_a_wave(h, w, layers):
    run_chain(h + layers, 1, h, w, layers)
    run_chain(h + layers + 1, 2, h, w, layers, top=255)
    run_chain(h + layers + 2, 1, h, w, layers, wide_shift=True)
