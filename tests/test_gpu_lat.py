"""GPU parity of the few-pixel convolution kernel (the waves of a workgroup split the K axis straight from global memory) against the
oracle, bit for bit: the library's own choice at these sizes, and forced where it would choose another kernel."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[False, True], ids=["chosen", "forced"])
def lat(request):
    from paper_2006_11735_amd import binding as B
    if request.param:
        B.icnn_set_tuning("lat", 1)
    yield
    B.icnn_set_tuning("reset")


def check(seed, n, h, w, cin, cout, k, stride=1, top=127, **kw):
    from gpu_util import gpu_conv2d
    g = np.random.default_rng(seed)
    x = g.integers(0, top + 1, size=(n, h, w, cin), dtype=np.uint8)
    wt = g.integers(-127, 128, size=(cout, k, k, cin), dtype=np.int8)
    b = g.integers(-4096, 4097, size=cout).astype(np.int32)
    ho, wo = (h + 2 * (k // 2) - k) // stride + 1, (w + 2 * (k // 2) - k) // stride + 1
    res = kw.pop("res_kind", None)
    if res == "u8":
        kw.update(res=g.integers(0, 128, size=(n, ho, wo, cout), dtype=np.uint8), res_mul=20000, res_shift=6)
    if res == "s32":
        kw.update(res=g.integers(-200000, 200000, size=(n, ho, wo, cout)).astype(np.int32), res_mul=20000, res_shift=15)
    kw.setdefault("mul", 20000)
    kw.setdefault("shift", 25)
    want = O.conv2d(x, wt, b, stride=stride, pad=k // 2, **kw)
    got = gpu_conv2d(x, wt, b, stride=stride, pad=k // 2, **kw)
    assert want.max() > want.min() and (got == want).all()


@pytest.mark.parametrize("shape", [
    (1, 7, 7, 512, 512, 3), (1, 7, 7, 2048, 64, 1), (3, 7, 7, 96, 40, 3), (1, 14, 14, 256, 1000, 1), (2, 9, 5, 128, 33, 3, 2), (1, 1, 1, 2048, 1000, 1),
    (33, 1, 1, 512, 96, 1), (1, 32, 1, 128, 32, 3), (1, 33, 1, 128, 32, 3), (1, 14, 14, 64, 128, 1, 2),
], ids=lambda s: "x".join(map(str, s)))
def test_shapes(lat, shape):
    check(sum(shape), *shape)


@pytest.mark.parametrize("name", ["no_fc", "no_lat"])
def test_the_classifier_off_this_kernel(name):
    from paper_2006_11735_amd import binding as B
    B.icnn_set_tuning(name, 1)
    try:
        check(21, 9, 1, 1, 512, 1000, 1, out_mode="raw_s32")
        check(22, 64, 1, 1, 2048, 40, 1)
    finally:
        B.icnn_set_tuning("reset")


@pytest.mark.parametrize("shape", [(1, 32, 32, 128, 512, 1), (1, 33, 32, 128, 512, 1), (10, 7, 7, 512, 512, 3), (11, 7, 7, 512, 512, 3), (10, 14, 14, 256, 256, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_on_either_side_of_what_is_on_the_chip_at_once(shape):
    # 512 and 528 work units; 256 and 272 where the kernel that splits K over a patch is nearer; 496 where it is not
    check(sum(shape), *shape)


def test_skip_operands_modes_and_inputs(lat):
    check(1, 1, 9, 9, 128, 64, 3, res_kind="u8", res_mode="pre")
    check(2, 1, 9, 9, 128, 64, 3, res_kind="u8", res_mode="post")
    check(3, 1, 9, 9, 128, 48, 3, res_kind="s32", res_mode="pre")
    check(4, 1, 9, 9, 128, 64, 3, out_mode="raw_s32")
    check(5, 1, 9, 9, 128, 64, 3, out_mode="linear_s8")
    check(6, 1, 9, 9, 128, 64, 3, out_mode="clamp_u8", lo=3, hi=200)
    check(7, 1, 9, 9, 128, 64, 3, top=255)
    check(8, 1, 9, 9, 128, 64, 3, mul=(1 << 30) + 1, shift=41)


def test_per_channel_parameters(lat):
    g = np.random.default_rng(9)
    for cout in (64, 40):
        pc = dict(mul_c=g.integers(1 << 14, 1 << 15, size=cout).astype(np.int32), shift_c=g.integers(23, 27, size=cout).astype(np.int32),
                  res_mul_c=g.integers(1 << 14, 1 << 15, size=cout).astype(np.int32), res_shift_c=g.integers(4, 9, size=cout).astype(np.int32))
        x = g.integers(0, 128, size=(1, 9, 9, 128), dtype=np.uint8)
        wt = g.integers(-127, 128, size=(cout, 3, 3, 128), dtype=np.int8)
        b = g.integers(-4096, 4097, size=cout).astype(np.int32)
        res = g.integers(0, 128, size=(1, 9, 9, cout), dtype=np.uint8)
        from gpu_util import gpu_conv2d
        want = O.conv2d(x, wt, b, pad=1, res=res, res_mode="pre", **pc)
        got = gpu_conv2d(x, wt, b, pad=1, res=res, res_mode="pre", **pc)
        assert (got == want).all()


@pytest.mark.parametrize("per_channel", [False, True])
def test_projection_block(lat, per_channel):
    # a block's last layer with its stride-2 projection: odd sizes, a channel count that is no multiple of 32
    import torch
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng(11)
    n, h, cm, cp, cout = 2, 5, 64, 96, 80
    xm = g.integers(0, 128, size=(n, h, h, cm), dtype=np.uint8)
    xp = g.integers(0, 128, size=(n, 2 * h - 1, 2 * h - 1, cp), dtype=np.uint8)
    wm = g.integers(-127, 128, size=(cout, 1, 1, cm), dtype=np.int8)
    wp = g.integers(-127, 128, size=(cout, 1, 1, cp), dtype=np.int8)
    bm, bp = (g.integers(-4096, 4097, size=cout).astype(np.int32) for _ in range(2))
    sk = O.conv2d(xp, wp, bp, stride=2, out_mode="raw_s32")
    pc = {}
    if per_channel:
        pc = dict(mul_c=g.integers(1 << 14, 1 << 15, size=cout).astype(np.int32), shift_c=g.integers(22, 25, size=cout).astype(np.int32),
                  res_mul_c=g.integers(1 << 14, 20000, size=cout).astype(np.int32), res_shift_c=np.full(cout, 15, np.int32))
    want = O.conv2d(xm, wm, bm, mul=20000, shift=23, res=sk, res_mode="pre", res_mul=20000, res_shift=15, **pc)
    dm = B.conv_desc(n=n, h=h, w=h, cin=cm, in_c_stride=cm, cout=cout, kh=1, kw=1, out_c_stride=cout, mul=20000, shift=23, res_mode=B.ICNN_RES_PRE,
                     res_dtype=B.ICNN_S32, res_c_stride=cout, res_mul=20000, res_shift=15)
    dp = B.conv_desc(n=n, h=2 * h - 1, w=2 * h - 1, cin=cp, in_c_stride=cp, cout=cout, kh=1, kw=1, stride_h=2, stride_w=2, out_c_stride=cout,
                     out_mode=B.ICNN_OUT_RAW_S32)
    packs = []
    for d, wt in ((dm, wm), (dp, wp)):
        packs.append(torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0"))
        B.iconv2d_prepack_weights(d, dev(wt), packs[-1])
    y = torch.zeros((n, h, h, cout), dtype=torch.uint8, device="cuda:0")
    if per_channel:
        arrs = [dev(pc[k]) for k in ("mul_c", "shift_c", "res_mul_c", "res_shift_c")]
        pcp = torch.zeros(B.iconv2d_packed_channel_params_bytes(dm), dtype=torch.uint8, device="cuda:0")
        B.iconv2d_prepack_channel_params(dm, B.channel_params(*arrs), pcp)
        B.iconv2d_dual_brelu_pc(dm, dev(xm), packs[0], dev(bm), pcp, dp, dev(xp), packs[1], dev(bp), y)
    else:
        B.iconv2d_dual_brelu(dm, dev(xm), packs[0], dev(bm), dp, dev(xp), packs[1], dev(bp), y)
    torch.cuda.synchronize()
    assert want.max() > 0 and (y.cpu().numpy() == want).all()
