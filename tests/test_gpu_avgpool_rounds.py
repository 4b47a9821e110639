"""Global average pool at the edges of its rounds of 64 positions (four waves, sixteen loads each) and of its 256 channels, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hw", [(1, 1), (1, 3), (2, 2), (1, 5), (3, 5), (7, 7), (7, 9), (8, 8), (5, 13), (1, 127), (3, 43)], ids=str)
@pytest.mark.parametrize("c", [4, 252, 256, 260])
def test_rounds(hw, c):
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    h, w = hw
    g = np.random.default_rng(h * w + c)
    x = g.integers(0, 256, size=(3, h, w, c), dtype=np.uint8)
    x[1] = 255
    mul = 32768 // (h * w)
    out = torch.full((3, c), 99, dtype=torch.uint8, device="cuda:0")
    B.iavgpool_global_u8(3, h, w, c, mul, 15, 255, dev(x), out)
    torch.cuda.synchronize()
    want = O.avgpool_global(x, mul, 15, 255)
    assert (out.cpu().numpy() == want.reshape(3, c)).all() and want.max() > 200
