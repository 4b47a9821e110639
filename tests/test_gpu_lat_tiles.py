"""GPU parity of the few-pixel kernel's tiles (16 x 16, 32 x 16, 32 x 32) and of its ways to place an activation fragment: pointwise, 3x3 from
arguments in registers, any window by steps of 64 channels, any multiple of 16 channels lane by lane.  Integers: bit for bit."""
import numpy as np
import pytest

from oracle import oracle as O
from test_gpu_lat import check

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[2, 3, 4], ids=["16x16", "32x16", "32x32"])
def tile(request):
    from paper_2006_11735_amd import binding as B
    B.icnn_set_tuning("lat", request.param)
    yield request.param
    B.icnn_set_tuning("reset")


# n, h, w, cin, cout, k[, stride]: remainders of pixels (15, 17, 33) and channels (8, 40), more waves than steps, more steps than are in flight
@pytest.mark.parametrize("shape", [
    (1, 1, 15, 64, 32, 1), (1, 3, 11, 128, 40, 1), (1, 17, 1, 64, 8, 1), (1, 2, 9, 6144, 32, 1),
    (1, 1, 1, 64, 16, 3), (2, 5, 7, 64, 48, 3), (1, 9, 13, 192, 40, 3, 2), (3, 7, 7, 512, 64, 3), (1, 6, 5, 1024, 32, 3),
    (1, 9, 9, 128, 40, 1, 2), (2, 6, 7, 64, 24, 5), (1, 8, 8, 64, 32, 5, 3), (1, 3, 200, 64, 32, 7),
    (1, 5, 7, 16, 40, 3), (2, 4, 9, 48, 32, 3), (1, 7, 5, 80, 24, 3, 2), (1, 33, 1, 112, 40, 1), (1, 9, 9, 32, 16, 5, 2), (1, 2, 3, 1040, 32, 3),
], ids=lambda s: "x".join(map(str, s)))
def test_edges(tile, shape):
    check(sum(shape), *shape)
    check(sum(shape) + 1, *shape, top=255, res_kind="u8", res_mode="pre")


def test_many_pixels_divide_lane_by_lane(tile):
    check(5, 2, 130, 127, 64, 16, 3)                          # 33020 pixels: beyond the divisions by one product


def test_epilogues(tile):
    check(1, 1, 9, 9, 128, 40, 1, res_kind="s32", res_mode="pre")
    check(2, 1, 9, 9, 128, 40, 3, res_kind="u8", res_mode="post")
    check(3, 1, 9, 9, 64, 40, 3, out_mode="raw_s32")
    check(4, 1, 9, 9, 64, 40, 3, out_mode="clamp_u8", lo=3, hi=200, mul=(1 << 30) + 1, shift=41)


# main and projection channels: steps within taps and lane by lane, the waves' shares at both ends
@pytest.mark.parametrize("cm,cp,cout", [(64, 128, 80), (512, 64, 40), (64, 1024, 32), (48, 80, 72)])
def test_projection_shares_the_waves(tile, cm, cp, cout):
    import torch
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng(cm + cp)
    n, h = 2, 5
    xm = g.integers(0, 128, size=(n, h, h, cm), dtype=np.uint8)
    xp = g.integers(0, 128, size=(n, 2 * h - 1, 2 * h - 1, cp), dtype=np.uint8)
    wm, wp = (g.integers(-127, 128, size=(cout, 1, 1, c), dtype=np.int8) for c in (cm, cp))
    bm, bp = (g.integers(-4096, 4097, size=cout).astype(np.int32) for _ in range(2))
    sk = O.conv2d(xp, wp, bp, stride=2, out_mode="raw_s32")
    want = O.conv2d(xm, wm, bm, mul=20000, shift=24, res=sk, res_mode="pre", res_mul=20000, res_shift=15)
    dm = B.conv_desc(n=n, h=h, w=h, cin=cm, in_c_stride=cm, cout=cout, kh=1, kw=1, out_c_stride=cout, mul=20000, shift=24, res_mode=B.ICNN_RES_PRE,
                     res_dtype=B.ICNN_S32, res_c_stride=cout, res_mul=20000, res_shift=15)
    dp = B.conv_desc(n=n, h=2 * h - 1, w=2 * h - 1, cin=cp, in_c_stride=cp, cout=cout, kh=1, kw=1, stride_h=2, stride_w=2, out_c_stride=cout,
                     out_mode=B.ICNN_OUT_RAW_S32)
    packs = []
    for d, wt in ((dm, wm), (dp, wp)):
        packs.append(torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0"))
        B.iconv2d_prepack_weights(d, dev(wt), packs[-1])
    y = torch.zeros((n, h, h, cout), dtype=torch.uint8, device="cuda:0")
    B.iconv2d_dual_brelu(dm, dev(xm), packs[0], dev(bm), dp, dev(xp), packs[1], dev(bp), y)
    torch.cuda.synchronize()
    assert want.max() > want.min() and (y.cpu().numpy() == want).all()
