"""Fused launches with requantisation per output channel: the same bytes as the layers one by one (iconv2d_brelu_pc, itself checked against
the oracle), over the forms that the packed parameters distinguish."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FORMS = ["plain", "mixed", "wide_skip"]


class Layer:
    def __init__(self, g, n, h, w, cin, cout, k=1, skip=None, form="plain", gain=1.0, cbuf=None):
        from gpu_util import dev
        from paper_2006_11735_amd import binding as B
        self.d = B.conv_desc(n=n, h=h, w=w, cin=cin, in_c_stride=cin, cout=cout, kh=k, kw=k, pad_h=k // 2, pad_w=k // 2, out_c_stride=cbuf or cout,
                             mul=1, shift=0, bound_q=127)
        w_ = g.integers(-127, 128, size=(cout, k, k, cin), dtype=np.int8)
        self.wp = torch.zeros(B.iconv2d_packed_weight_bytes(self.d), dtype=torch.uint8, device="cuda:0")
        B.iconv2d_prepack_weights(self.d, dev(w_), self.wp)
        self.bias = dev(g.integers(-4096, 4097, size=cout).astype(np.int32))
        # a ratio per channel that leaves most results inside the clamp: 127 / (about three standard deviations of the sums)
        ratio = gain * 127.0 / (3 * 73 * 64 * np.sqrt(cin * k * k)) * g.uniform(0.5, 2.0, size=cout)
        shift = g.integers(22, 27, size=cout)
        if form in FORMS[1:]:                        # shifts beyond 32 and, now and then, a ratio above one half
            shift = np.where(np.arange(cout) % 3 == 0, g.integers(33, 40, size=cout), shift)
            ratio = np.where(np.arange(cout) % 17 == 5, 1.5, ratio)
        mul = np.clip(np.round(ratio * 2.0 ** shift), 1, 2 ** 31 - 1)
        arrs = [mul, shift]
        if skip is not None:
            self.d.res_mode, self.d.res_dtype, self.d.res_c_stride = B.ICNN_RES_PRE, B.ICNN_U8 if skip == "u8" else B.ICNN_S32, cout
            rs = g.integers(25, 28, size=cout) if form == "wide_skip" else g.integers(3, 8, size=cout)
            rr = g.uniform(200, 400, size=cout) if skip == "u8" else g.uniform(0.5, 1.4, size=cout)
            if skip != "u8":
                rs = rs + 10
            arrs += [np.minimum(np.round(rr * 2.0 ** rs), 2 ** 31 - 1), rs]
            if form not in FORMS and skip == "u8":   # rescales that are one product each: shifts 0 to 30, the largest multipliers among them
                rs = g.integers(0, 31, size=cout)
                top = (2 ** 31 - 1 - ((1 << rs) >> 1)) // 255
                arrs[2:] = [np.where(np.arange(cout) % 5 == 0, top, np.minimum(np.round(rr * 2.0 ** rs), top)), rs]
            self.d.res_mul, self.d.res_shift = (1, 0) if skip == "u8" else (3, 1)
        at = cout - 7                                # one channel of the last group, or none, that is not one product
        if form == "one factor":
            arrs[1][at] = 33
        elif form == "one shift" and skip == "u8":
            arrs[3][at] = 31
        elif form == "one multiplier" and skip == "u8":
            arrs[2][at] = 2 ** 31 - 1
        self.pc = torch.zeros(B.iconv2d_packed_channel_params_bytes(self.d), dtype=torch.uint8, device="cuda:0")
        keep = [dev(a.astype(np.int32)) for a in arrs]
        B.iconv2d_prepack_channel_params(self.d, B.channel_params(*keep), self.pc)
        torch.cuda.synchronize()

    def run(self, x, res=None):
        from paper_2006_11735_amd import binding as B
        d = self.d
        y = torch.zeros((d.n, d.h, d.w, d.out_c_stride), dtype=torch.uint8, device="cuda:0")
        B.iconv2d_brelu_pc(d, x, self.wp, self.bias, self.pc, res, y, None)
        return y


def picture(g, *shape):
    return torch.from_numpy(g.integers(0, 128, size=shape, dtype=np.uint8)).cuda()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("shape", [(2, 56, 56, 256), (1, 17, 23, 128), (1, 5, 6, 64), (12, 56, 56, 256)], ids=lambda s: "x".join(map(str, s)))
def test_bottleneck_block(shape, form):
    from paper_2006_11735_amd import binding as B
    n, h, w, c = shape
    g = np.random.default_rng(sum(shape))
    x = picture(g, n, h, w, c)
    for skip in ("u8", None):
        l1, l2, l3 = Layer(g, n, h, w, c, 64, form=form), Layer(g, n, h, w, 64, 64, 3, form=form), Layer(g, n, h, w, 64, c, skip=skip, form=form)
        res = x if skip else None
        want = l3.run(l2.run(l1.run(x)), res)
        got = torch.zeros_like(want)
        B.iconv2d_bottleneck_brelu_pc(l1.d, x, l1.wp, l1.bias, l1.pc, l2.d, l2.wp, l2.bias, l2.pc, l3.d, l3.wp, l3.bias, l3.pc, res, got)
        assert torch.equal(got, want), (skip, int((got != want).sum()))
        assert 3 < len(torch.unique(want))


# one product per output with the skip operand, in the waves all of whose channels allow it: all of them, all but the last group's
@pytest.mark.parametrize("form", ["products", "one factor", "one shift", "one multiplier"])
@pytest.mark.parametrize("shape", [(1, 17, 23, 256), (1, 9, 14, 128), (2, 5, 6, 64)], ids=lambda s: "x".join(map(str, s)))
def test_bottleneck_block_with_a_channel_of_another_form(shape, form):
    test_bottleneck_block(shape, form)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("shape", [(2, 56, 56), (1, 9, 31)], ids=lambda s: "x".join(map(str, s)))
def test_bottleneck_block_with_projection(shape, form):
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    n, h, w = shape
    g = np.random.default_rng(sum(shape))
    x = picture(g, n, h, w, 64)
    l1, l2, l3 = Layer(g, n, h, w, 64, 64, form=form), Layer(g, n, h, w, 64, 64, 3, form=form), Layer(g, n, h, w, 64, 256, skip="s32", form=form)
    dp = B.conv_desc(n=n, h=h, w=w, cin=64, in_c_stride=64, cout=256, kh=1, kw=1, out_c_stride=256, out_mode=B.ICNN_OUT_RAW_S32)
    wp = torch.zeros(B.iconv2d_packed_weight_bytes(dp), dtype=torch.uint8, device="cuda:0")
    B.iconv2d_prepack_weights(dp, dev(g.integers(-127, 128, size=(256, 1, 1, 64), dtype=np.int8)), wp)
    bp = dev(g.integers(-4096, 4097, size=256).astype(np.int32))
    skip = torch.zeros((n, h, w, 256), dtype=torch.int32, device="cuda:0")
    B.iconv2d_brelu(dp, x, wp, bp, None, skip, None)
    want = l3.run(l2.run(l1.run(x)), skip)
    got = torch.zeros_like(want)
    B.iconv2d_bottleneck_dual_brelu_pc(l1.d, x, l1.wp, l1.bias, l1.pc, l2.d, l2.wp, l2.bias, l2.pc, l3.d, l3.wp, l3.bias, l3.pc, dp, wp, bp, got)
    assert torch.equal(got, want), int((got != want).sum())
    assert 3 < len(torch.unique(want))


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("shape", [(4, 14, 14, 256, 1024), (2, 28, 28, 128, 512), (1, 1, 1, 64, 256), (3, 5, 9, 128, 768)],
                         ids=lambda s: "x".join(map(str, s)))
def test_pair(shape, form):
    from paper_2006_11735_amd import binding as B
    n, h, w, mid, c = shape
    g = np.random.default_rng(sum(shape))
    t, res = picture(g, n, h, w, mid), picture(g, n, h, w, c)
    for skip in ("u8", None):
        l3, l1 = Layer(g, n, h, w, mid, c, skip=skip, form=form), Layer(g, n, h, w, c, mid, form=form)
        y = l3.run(t, res if skip else None)
        z = l1.run(y)
        gy, gz = torch.zeros_like(y), torch.zeros_like(z)
        B.iconv2d_pair_brelu_pc(l3.d, t, l3.wp, l3.bias, l3.pc, res if skip else None, gy, l1.d, l1.wp, l1.bias, l1.pc, gz)
        assert torch.equal(gy, y) and torch.equal(gz, z), skip


@pytest.mark.parametrize("form", FORMS[:2])
@pytest.mark.parametrize("cout", [32, 64])
def test_first_layer_with_pool(cout, form):
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng(cout)
    n, h, w = 2, 61, 75
    l = Layer(g, n, h, w, 3, cout, 7, form=form)
    d = l.d
    d.stride_h = d.stride_w = 2
    x = picture(g, n, h, w, 3)
    ho, wo = B.iconv2d_out_hw(d)
    t = torch.zeros((n, ho, wo, cout), dtype=torch.uint8, device="cuda:0")
    ws = torch.zeros(B.iconv2d_workspace_bytes(d), dtype=torch.uint8, device="cuda:0")
    B.iconv2d_brelu_pc(d, x, l.wp, l.bias, l.pc, None, t, ws)
    hp, wp = (ho - 1) // 2 + 1, (wo - 1) // 2 + 1
    want = torch.zeros((n, hp, wp, cout), dtype=torch.uint8, device="cuda:0")
    B.imaxpool2d_u8(n, ho, wo, cout, 3, 2, 1, t, want)
    got = torch.zeros_like(want)
    B.iconv2d_maxpool_brelu_pc(d, 3, 2, 1, x, l.wp, l.bias, l.pc, got)
    assert torch.equal(got, want)
    assert 3 < len(torch.unique(want))


def test_refused_shapes_launch_nothing():
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng(0)
    x = picture(g, 1, 8, 8, 512)
    l1, l2, l3 = Layer(g, 1, 8, 8, 512, 128), Layer(g, 1, 8, 8, 128, 128, 3), Layer(g, 1, 8, 8, 128, 512, skip="u8")
    y = torch.full((1, 8, 8, 512), 7, dtype=torch.uint8, device="cuda:0")
    with pytest.raises(B.IcnnError) as e:            # 128 middle channels
        B.iconv2d_bottleneck_brelu_pc(l1.d, x, l1.wp, l1.bias, l1.pc, l2.d, l2.wp, l2.bias, l2.pc, l3.d, l3.wp, l3.bias, l3.pc, x, y)
    assert e.value.code == B.ICNN_E_UNSUPPORTED
    a, b = Layer(g, 1, 8, 8, 256, 2048), Layer(g, 1, 8, 8, 2048, 256)
    with pytest.raises(B.IcnnError) as e:            # parameters of 2048 channels beside the tile
        B.iconv2d_pair_brelu_pc(a.d, x, a.wp, a.bias, a.pc, None, y, b.d, b.wp, b.bias, b.pc, y)
    assert e.value.code == B.ICNN_E_UNSUPPORTED
    assert (y == 7).all()
