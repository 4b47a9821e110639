"""The 3x3 and 1x1 kernel of strides 1 and 2 whose weights go straight into registers (iconv2d_brelu, iconv2d_brelu_pc), at the edges of its tiles and in
every form it takes, against the oracle; and the library's choice against the kernel it would take otherwise."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture
def flat():
    from paper_2006_11735_amd import binding as B
    B.icnn_set_tuning("flat", 1)
    yield
    B.icnn_set_tuning("reset")


def layer(seed, n, h, w, cin, cout, k, pitch=0, signed=False):
    g = np.random.default_rng(seed)
    shape = (n, h, w, cin + pitch)
    x = g.integers(-128, 128, size=shape).astype(np.int8) if signed else g.integers(0, 128, size=shape).astype(np.uint8)
    wt = g.integers(-127, 128, size=(cout, k, k, cin), dtype=np.int8)
    return g, x, wt, g.integers(-4096, 4097, size=cout).astype(np.int32)


def check(x, wt, b, **kw):
    from gpu_util import gpu_conv2d
    kw.setdefault("mul", 20000)
    kw.setdefault("shift", 25)
    got = gpu_conv2d(x, wt, b, pad=wt.shape[1] // 2, **kw)
    kw.pop("misalign", None)
    want = O.conv2d(x, wt, b, pad=wt.shape[1] // 2, cin=wt.shape[3], **kw)
    assert want.max() > want.min() and (got == want).all()


# one pixel, one row, one column, a last tile of one pixel, of 63, pictures smaller and larger than a tile, every channel count it is built for
@pytest.mark.parametrize("shape", [(1, 1, 1, 64, 64, 3), (1, 1, 129, 64, 64, 3), (1, 65, 1, 128, 128, 3), (3, 5, 13, 64, 128, 3), (5, 7, 7, 512, 128, 3),
                                   (2, 14, 14, 256, 256, 3), (1, 9, 47, 256, 128, 3), (1, 3, 200, 64, 64, 3), (127, 1, 1, 256, 128, 1), (1, 1, 1, 512, 256, 1),
                                   (1, 13, 5, 1024, 128, 1), (2, 8, 8, 1024, 384, 1), (1, 2, 2, 128, 128, 3), (300, 2, 3, 64, 64, 3),
                                   (1, 5, 13, 2048, 128, 1), (1, 63, 1, 128, 128, 1)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("skip", [False, True], ids=["plain", "skip"])
def test_tiles(flat, shape, skip):
    g, x, wt, b = layer(sum(shape), *shape)
    kw = dict(res=g.integers(0, 128, size=shape[:3] + shape[4:5], dtype=np.uint8), res_mode="pre", res_mul=20000, res_shift=5) if skip else {}
    check(x, wt, b, mul=32767, shift=25, **kw)


# stride 2: one pixel, even and odd pictures, rows and columns of one, pictures smaller and larger than a tile
@pytest.mark.parametrize("shape", [(1, 1, 1, 64, 128, 3), (3, 7, 9, 64, 128, 3), (2, 28, 28, 256, 128, 3), (5, 8, 7, 128, 128, 3), (1, 1, 131, 128, 128, 3),
                                   (1, 131, 1, 64, 256, 3), (9, 2, 2, 256, 128, 3), (6, 14, 14, 512, 128, 3), (130, 1, 1, 128, 128, 3), (2, 13, 30, 64, 128, 1),
                                   (1, 9, 15, 128, 256, 1), (3, 7, 7, 256, 128, 1), (1, 17, 17, 512, 128, 1)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("form", ["plain", "skip", "raw", "per channel"])
def test_stride_2(flat, shape, form):
    from test_gpu_conv import channel_params
    g, x, wt, b = layer(sum(shape), *shape)
    n, h, w = shape[:3]
    res = g.integers(0, 128, size=(n, (h + 1) // 2, (w + 1) // 2, shape[4]), dtype=np.uint8)
    check(x, wt, b, stride=2, **{"plain": {}, "skip": dict(res=res, res_mode="pre", res_mul=20000, res_shift=5), "raw": dict(out_mode="raw_s32"),
                                 "per channel": channel_params(3, shape[4])}[form])


@pytest.mark.parametrize("kw", [dict(out_mode="raw_s32"), dict(out_mode="linear_s8"), dict(out_mode="clamp_u8", lo=3, hi=250), dict(bound_q=15), dict(mul=20001, shift=24),
                                dict(mul=2**31 - 1, shift=43), dict(mul=1, shift=9)], ids=str)
@pytest.mark.parametrize("res", [None, "u8", "s8", "s32", "post"])
@pytest.mark.parametrize("shape", [(1, 9, 11, 64, 64, 3), (1, 9, 11, 256, 128, 1)], ids=lambda s: "x".join(map(str, s)))
def test_modes(flat, shape, res, kw):
    g, x, wt, b = layer(5, *shape)
    out = shape[:3] + shape[4:5]
    if res == "post" and kw.get("out_mode") == "raw_s32":
        res = "u8"                     # a raw accumulator has no requantised output to add to
    r = {None: None, "u8": g.integers(0, 128, size=out, dtype=np.uint8), "post": g.integers(0, 128, size=out, dtype=np.uint8),
         "s8": g.integers(-128, 128, size=out).astype(np.int8), "s32": g.integers(-300000, 300000, size=out).astype(np.int32)}[res]
    more = {} if r is None else dict(res=r, res_mode="post" if res == "post" else "pre", res_mul=20000, res_shift=15 if res == "s32" else 5)
    check(x, wt, b, **{**kw, **more})


def test_inputs_pitches_and_channel_parameters(flat):
    from test_gpu_conv import channel_params
    for shape in ((1, 10, 11, 128, 128, 3), (2, 6, 6, 512, 128, 1)):
        g, x, wt, b = layer(7, *shape, pitch=48)
        res = g.integers(0, 128, size=shape[:3] + shape[4:5], dtype=np.uint8)
        check(x, wt, b, out=np.zeros(shape[:3] + (shape[4] + 48,), np.uint8), out_c_offset=32)
        check(x, wt, b, misalign=1)                      # unaligned addresses stay on a kernel that takes them
        check(x, wt, b, res=res, res_mode="pre", **channel_params(8, shape[4], res=True))
        check(x, wt, b, out_mode="linear_s8", **channel_params(9, shape[4]))
        _g, x, wt, b = layer(10, *shape, signed=True)
        check(x, wt, b)
        check(x.view(np.uint8), wt, b)                   # bytes up to 255


# per channel: factors and skip rescales that are one product each (shifts 0 to 30, the largest multipliers among them), and a last wave where one is not
@pytest.mark.parametrize("odd", [None, "factor", "shift", "multiplier"])
@pytest.mark.parametrize("shape", [(1, 9, 11, 64, 64, 3), (1, 9, 11, 256, 256, 1), (2, 7, 9, 128, 128, 3)], ids=lambda s: "x".join(map(str, s)))
def test_per_channel_products(flat, shape, odd):
    g, x, wt, b = layer(12, *shape)
    cout = shape[4]
    rs = g.integers(0, 31, size=cout)
    rm = np.where(np.arange(cout) % 5 == 0, (2**31 - 1 - ((1 << rs) >> 1)) // 255, g.integers(1, 1 << 15, size=cout))
    pc = dict(mul_c=g.integers(1 << 14, 1 << 15, size=cout).astype(np.int32), shift_c=g.integers(21, 33, size=cout).astype(np.int32),
              res_mul_c=rm.astype(np.int32), res_shift_c=rs.astype(np.int32))
    if odd:
        name, value = {"factor": ("shift_c", 33), "shift": ("res_shift_c", 31), "multiplier": ("res_mul_c", 2**31 - 1)}[odd]
        pc[name][cout - 7] = value
    res = g.integers(0, 256, size=shape[:4][:3] + (cout,), dtype=np.uint8)
    check(x, wt, b, res=res, res_mode="pre", **pc)
    check(x, wt, b, res=res, res_mode="pre", out_mode="linear_s8", **pc)
    check(x, wt, b, mul_c=pc["mul_c"], shift_c=pc["shift_c"])


# rescales of the skip operand's 255 on both sides of int32, by the library's own choice of kernel.  The output's ratio is 2^-24, so that a
# sum's top bits are what is stored; (255 * 16777215 / 2 is an int32, twice that is not)
@pytest.mark.parametrize("rescale", [(8421504, 0), (8421505, 0), (10000000, 0), (16777215, 0), (16777215, 1), (2**31 - 1, 0)], ids=str)
@pytest.mark.parametrize("shape", [(1, 46, 46, 128, 128, 1), (1, 70, 60, 64, 64, 3), (1, 46, 46, 128, 128, 3)], ids=lambda s: "x".join(map(str, s)))
def test_skip_rescales_at_the_end_of_int32(shape, rescale):
    g, x, wt, b = layer(13, *shape)
    res = g.integers(0, 256, size=shape[:3] + shape[4:5], dtype=np.uint8)
    res[0, 5:9] = 255
    check(x, wt, b, res=res, res_mode="pre", res_mul=rescale[0], res_shift=rescale[1], mul=1, shift=24)


@pytest.mark.parametrize("shape", [(6, 14, 14, 256, 256, 3), (5, 14, 14, 256, 256, 3), (17, 7, 7, 512, 512, 3), (3, 28, 28, 128, 128, 3), (2, 28, 28, 512, 128, 1),
                                   (9, 14, 14, 1024, 256, 1), (2, 56, 56, 64, 64, 3), (2, 30, 30, 256, 1024, 1), (16, 7, 7, 2048, 512, 1), (90, 7, 7, 2048, 512, 1)], ids=lambda s: "x".join(map(str, s)))
def test_the_librarys_choice(shape):
    # on either side of 256 units of 32 channels x 32 pixels, with and without a skip operand
    from gpu_util import gpu_conv2d
    from paper_2006_11735_amd import binding as B
    g, x, wt, b = layer(11, *shape)
    res = g.integers(0, 128, size=shape[:3] + shape[4:5], dtype=np.uint8)
    for kw in ({}, dict(res=res, res_mode="pre", res_mul=20000, res_shift=5)):
        got = []
        for how in (0, 1, 2):
            B.icnn_set_tuning("flat", how)
            try:
                got.append(gpu_conv2d(x, wt, b, pad=shape[5] // 2, mul=20000, shift=25, **kw))
            finally:
                B.icnn_set_tuning("reset")
        assert got[0].max() > 0 and (got[0] == got[1]).all() and (got[0] == got[2]).all()


# one tile, one pixel, the last tile of one pixel and of 63, strides 1 and 2 on even and odd pictures, every channel count it is built for
@pytest.mark.parametrize("shape", [(1, 1, 1, 128, 128, 2), (1, 13, 5, 128, 256, 2), (3, 7, 9, 256, 128, 2), (1, 9, 7, 512, 128, 1), (127, 1, 1, 256, 128, 1),
                                   (1, 1, 130, 128, 128, 2), (5, 7, 7, 512, 384, 2), (9, 14, 14, 256, 256, 1)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("form", ["plain", "wide", "s8", "per channel"])
def test_closing_layer_with_projection(shape, form):
    import torch
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    n, h, w, cm, cout, stride = shape
    hp, wp = h * stride, (w - 1) * stride + 1                               # at stride 2 even heights, odd widths
    g = np.random.default_rng(sum(shape))
    xm, xp = g.integers(0, 128, size=(n, h, w, cm), dtype=np.uint8), g.integers(0, 128, size=(n, hp, wp, 2 * cm), dtype=np.uint8)
    wm, wq = g.integers(-127, 128, size=(cout, 1, 1, cm), dtype=np.int8), g.integers(-127, 128, size=(cout, 1, 1, 2 * cm), dtype=np.int8)
    bm, bq = (g.integers(-4096, 4097, size=cout).astype(np.int32) for _ in range(2))
    kw = dict(mul=23187, shift=27, res_mul=20011, res_shift=15)
    if form == "wide":
        kw.update(mul=2**31 - 1, shift=43, res_mul=1, res_shift=0)
    if form == "s8":
        kw["out_mode"] = "linear_s8"
    pc = {}
    if form == "per channel":
        pc = dict(mul_c=g.integers(1 << 14, 1 << 15, size=cout).astype(np.int32), shift_c=g.integers(24, 29, size=cout).astype(np.int32),
                  res_mul_c=g.integers(1 << 14, 20011, size=cout).astype(np.int32), res_shift_c=g.integers(15, 17, size=cout).astype(np.int32))
    want = O.conv2d(xm, wm, bm, bound_q=127, res=O.conv2d(xp, wq, bq, stride=stride, out_mode="raw_s32"), res_mode="pre", **kw, **pc)
    out_mode = B.ICNN_OUT_LINEAR_S8 if form == "s8" else B.ICNN_OUT_BRELU_U8
    dm = B.conv_desc(n=n, h=h, w=w, cin=cm, in_c_stride=cm, cout=cout, kh=1, kw=1, out_c_stride=cout, mul=kw["mul"], shift=kw["shift"], bound_q=127, out_mode=out_mode,
                     res_mode=B.ICNN_RES_PRE, res_dtype=B.ICNN_S32, res_c_stride=cout, res_mul=kw["res_mul"], res_shift=kw["res_shift"])
    dp = B.conv_desc(n=n, h=hp, w=wp, cin=2 * cm, in_c_stride=2 * cm, cout=cout, kh=1, kw=1, stride_h=stride, stride_w=stride, out_c_stride=cout,
                     out_mode=B.ICNN_OUT_RAW_S32)
    packs = []
    for d, wt in ((dm, wm), (dp, wq)):
        packs.append(torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0"))
        B.iconv2d_prepack_weights(d, dev(wt), packs[-1])
    args = dev(xm), packs[0], dev(bm)
    if pc:
        arrs = [dev(pc[k]) for k in ("mul_c", "shift_c", "res_mul_c", "res_shift_c")]
        pcp = torch.zeros(B.iconv2d_packed_channel_params_bytes(dm), dtype=torch.uint8, device="cuda:0")
        B.iconv2d_prepack_channel_params(dm, B.channel_params(*arrs), pcp)
        args += (pcp,)
    other = dev(xp), packs[1], dev(bq)
    fn = B.iconv2d_dual_brelu_pc if pc else B.iconv2d_dual_brelu
    for name, value in (("no_lat", 1), ("flat", 2)):                        # this kernel, the others
        y = torch.full((n, h, w, cout), 99, dtype=torch.int8 if form == "s8" else torch.uint8, device="cuda:0")
        B.icnn_set_tuning(name, value)
        try:
            fn(dm, *args, dp, *other, y)
        finally:
            B.icnn_set_tuning("reset")
        assert want.max() > 0 and (y.cpu().numpy() == want).all()
