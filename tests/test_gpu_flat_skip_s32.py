"""3x3 layers that join an int32 skip operand before requantisation, in the kernel whose weights go straight into registers: operands up to both
ends of int32, rescales inside and outside the two-product form, against the oracle, bit for bit."""
import numpy as np
import pytest

from oracle import oracle as O
from test_gpu_flat import flat, layer  # noqa: F401  (flat: fixture)

pytestmark = pytest.mark.gpu

I32 = np.iinfo(np.int32)


def check(x, wt, b, **kw):
    # (a small ratio beside a small rescale stores one value everywhere: equality alone counts)
    from gpu_util import gpu_conv2d
    got = gpu_conv2d(x, wt, b, pad=1, **kw)
    assert (got == O.conv2d(x, wt, b, pad=1, cin=wt.shape[3], **kw)).all()


# shifts at both ends of the form's range and beyond them, multipliers up to the largest; the requantisation at the edge of what an overflow's
# remainder may change (mul / 2^shift of 2^-24 gives 127 or 128 at int32's end), and one that is not one product's high word
@pytest.mark.parametrize("rescale", [(21691, 4), (1, 2), (3, 2), (2**31 - 1, 2), (24547, 13), (2**31 - 1, 30), (12345, 30), (7, 1), (2**31 - 1, 31), (5, 0)], ids=str)
@pytest.mark.parametrize("ratio", [(29249, 26), (1, 24), (1, 23), (20000 << 14, 38), (30000, 15)], ids=str)
def test_rescales(flat, rescale, ratio):  # noqa: F811
    g, x, wt, b = layer(rescale[1] + ratio[1], 2, 7, 9, 64, 128, 3)
    res = g.integers(-40000, 40001, size=(2, 7, 9, 128)).astype(np.int32) >> g.integers(0, 16, size=(2, 7, 9, 128)).astype(np.int32)
    res[0, 0] = g.integers(I32.min, I32.max + 1, size=(9, 128))
    res[0, 1, 0], res[0, 1, 1] = I32.min, I32.max
    kw = dict(res=res, res_mode="pre", res_mul=rescale[0], res_shift=rescale[1], mul=ratio[0], shift=ratio[1])
    check(x, wt, b, **kw)
    check(x, wt, b, out_mode="clamp_u8", lo=3, hi=255, **kw)
    check(x, wt, b, out_mode="linear_s8", **kw)


@pytest.mark.parametrize("shape", [(1, 1, 1, 64, 128, 3), (1, 9, 47, 256, 128, 3), (3, 5, 13, 128, 256, 3), (5, 7, 7, 512, 128, 3), (1, 1, 65, 64, 256, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_tiles(flat, shape):  # noqa: F811
    g, x, wt, b = layer(sum(shape), *shape)
    res = g.integers(-500000, 500001, size=shape[:3] + shape[4:5]).astype(np.int32)
    check(x, wt, b, res=res, res_mode="pre", res_mul=24547, res_shift=13, mul=32767, shift=26)
    check(x, wt, b, res=res, res_mode="post", res_mul=24547, res_shift=28, mul=32767, shift=26)
