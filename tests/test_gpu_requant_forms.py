"""Every requantisation form of the convolution epilogues at the places where it can go wrong: accumulators on both sides of each rounding step
and of both clamps, against exact integers.  The input is zero, so channel c's accumulator is its bias."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def exact(t, mul, shift, hi):
    q = (int(t) * mul + ((1 << shift) >> 1)) >> shift
    return min(max(q, 0), hi)


@pytest.mark.parametrize("tile", [-1, 1, 4])
@pytest.mark.parametrize("mul, shift, hi", [
    (16385, 24, 127),            # product fits 32 bits
    (16385, 25, 255), (16385, 26, 127), (32767, 26, 127), (32767, 27, 255), (16385, 30, 127), (16385, 31, 255), (16385, 33, 3),   # its high half, 24-bit factors
    (32767, 23, 127),            # one bit more than the high half takes
    (16385, 34, 1), (1 << 23, 40, 7), ((1 << 30) + 1, 40, 127), (3, 1, 255), (1, 0, 255),
])
def test_rounding_steps_and_clamps(tile, mul, shift, hi):
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    steps = []
    for k in list(range(0, 5)) + list(range(max(0, hi - 3), hi + 3)):
        t = ((2 * k + 1) << shift) // (2 * mul)            # where [t mul / 2^shift] goes from k to k + 1
        steps += [t - 1, t, t + 1, t + 2]
    rng = np.random.default_rng(shift)
    top = ((2 * hi + 1) << shift) // (2 * mul) + 2
    steps += [-1, -5, -(1 << 30), 1 << 30] + [int(v) for v in rng.integers(-top, top + 1, size=64)]
    steps = [t for t in steps if abs(t) <= 1 << 30]
    cout = (len(steps) + 63) // 64 * 64
    bias = np.array(steps + [0] * (cout - len(steps)), dtype=np.int32)
    n = 200                                                # pixels: several tiles of every kernel
    d = B.conv_desc(n=1, h=n, w=1, cin=64, in_c_stride=64, cout=cout, kh=1, kw=1, out_c_stride=cout, mul=mul, shift=shift, bound_q=hi)
    wp = torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0")
    B.iconv2d_prepack_weights(d, dev(rng.integers(-127, 128, size=(cout, 1, 1, 64), dtype=np.int8)), wp)
    y = torch.zeros((n, cout), dtype=torch.uint8, device="cuda:0")
    B.icnn_set_tuning("tile", tile)
    try:
        B.iconv2d_brelu(d, torch.zeros((n, 64), dtype=torch.uint8, device="cuda:0"), wp, dev(bias), None, y)
        torch.cuda.synchronize()
    finally:
        B.icnn_set_tuning("reset")
    want = np.array([exact(t, mul, shift, hi) for t in bias], dtype=np.uint8)
    assert (y.cpu().numpy() == want[None, :]).all()
