"""A 3x3 layer, the 1x1 layer that closes its block and the 1x1 layer that opens the next one as one call (iconv2d_triple_brelu).  The fused kernel (a
forced tile): the same bytes as the three layers one by one, which have their own tests against the oracle, at the edges of tiles and images.  The
library's own choice, which takes the layers of small calls apart: against the oracle, on both sides of each of its conditions."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


class Layer:
    """A layer with weights and parameters on the GPU.  form: how it requantises: "rq24" a 15-bit multiplier (the 32-bit form), "hi" one that only
    the one-multiply form takes, "wide" a shift beyond 32; "pc", "pc_mixed" per channel (all channels plain; some not)."""

    def __init__(self, g, n, h, w, cin, cout, k=1, skip=False, form="rq24", pitch=None, in_pitch=None, rescale=(20000, 6)):
        from gpu_util import dev
        from paper_2006_11735_amd import binding as B
        ratio = 127.0 / (3 * 73 * 64 * np.sqrt(cin * k * k))
        shift = 14 + int(np.floor(-np.log2(ratio)))
        mul = int(round(ratio * 2.0 ** shift))
        if form == "hi":
            mul, shift = mul << 11, shift + 11
        elif form == "wide":
            mul, shift = mul << 12, shift + 12
        self.d = d = B.conv_desc(n=n, h=h, w=w, cin=cin, in_c_stride=in_pitch or cin, cout=cout, kh=k, kw=k, pad_h=k // 2, pad_w=k // 2,
                                 out_c_stride=pitch or cout, out_c_offset=0, mul=mul, shift=shift, bound_q=127)
        self.pc = None
        self.wp = torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0")
        self.w_host = g.integers(-127, 128, size=(cout, k, k, cin), dtype=np.int8)
        B.iconv2d_prepack_weights(d, dev(self.w_host), self.wp)
        self.bias_host = g.integers(-4096, 4097, size=cout).astype(np.int32)
        self.bias = dev(self.bias_host)
        if skip:
            d.res_mode, d.res_dtype, d.res_c_stride, d.res_mul, d.res_shift = (B.ICNN_RES_PRE, B.ICNN_U8, cout) + rescale
        if form.startswith("pc"):
            sh = g.integers(24, 29, size=cout)
            rt = ratio * g.uniform(0.5, 2.0, size=cout)
            if form == "pc_mixed":
                sh = np.where(np.arange(cout) % 3 == 0, g.integers(33, 38, size=cout), sh)
                rt = np.where(np.arange(cout) % 17 == 5, 1.5, rt)
            arrs = [np.clip(np.round(rt * 2.0 ** sh), 1, 2 ** 31 - 1), sh]
            if skip:
                arrs += [g.integers(15000, 30000, size=cout), g.integers(5, 8, size=cout)]
            keep = [dev(a.astype(np.int32)) for a in arrs]
            self.pc = torch.zeros(B.iconv2d_packed_channel_params_bytes(d), dtype=torch.uint8, device="cuda:0")
            B.iconv2d_prepack_channel_params(d, B.channel_params(*keep), self.pc)
        torch.cuda.synchronize()

    def run(self, x, res=None):
        from paper_2006_11735_amd import binding as B
        y = torch.full((self.d.n, self.d.h, self.d.w, self.d.out_c_stride), 99, dtype=torch.uint8, device="cuda:0")
        if self.pc is not None:
            B.iconv2d_brelu_pc(self.d, x, self.wp, self.bias, self.pc, res, y, None)
        else:
            B.iconv2d_brelu(self.d, x, self.wp, self.bias, res, y, None)
        return y


    def oracle(self, x, res=None):
        from oracle import oracle as O
        d = self.d
        skip = {} if res is None else dict(res=res, res_mode="pre", res_mul=d.res_mul, res_shift=d.res_shift)
        return O.conv2d(x, self.w_host, self.bias_host, pad=d.pad_h, mul=d.mul, shift=d.shift, bound_q=127, **skip)


def picture(g, *shape):
    return torch.from_numpy(g.integers(0, 128, size=shape, dtype=np.uint8)).cuda()


def check(n, h, w, form="rq24", skip=True, third=True, middle=True, pitches=(0, 0, 0), in_place=False, lanes=1, rescale=(20000, 6)):
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng([n, h, w])
    mid, wide = 256, 1024
    l2 = Layer(g, n, h, w, mid, mid, 3, form=form, pitch=mid + pitches[0])
    l3 = Layer(g, n, h, w, mid, wide, skip=skip, form=form, rescale=rescale, pitch=wide + pitches[1], in_pitch=mid + pitches[0])
    l1 = Layer(g, n, h, w, wide, mid, form=form, pitch=mid + pitches[2], in_pitch=wide + pitches[1])
    t = picture(g, n, h, w, mid)
    res = torch.from_numpy(g.integers(0, 256, size=(n, h, w, wide), dtype=np.uint8)).cuda() if skip else None
    b = l2.run(t)
    y = l3.run(b, res)
    z = l1.run(y)
    assert len(torch.unique(z)) > 3 and len(torch.unique(y)) > 3
    gb, gy, gz = (torch.full_like(q, 99) for q in (b, y, z))
    if in_place:
        gy = res.clone()
        res = gy
    tail = (l1.d, l1.wp, l1.bias) + ((l1.pc,) if l1.pc is not None else ()) + (gz,) if third else (None,) * (5 if l1.pc is not None else 4)
    if l2.pc is not None:
        B.iconv2d_triple_brelu_pc(l2.d, t, l2.wp, l2.bias, l2.pc, gb if middle else None, l3.d, l3.wp, l3.bias, l3.pc, res, gy, *tail, lanes=lanes)
    else:
        B.iconv2d_triple_brelu(l2.d, t, l2.wp, l2.bias, gb if middle else None, l3.d, l3.wp, l3.bias, res, gy, *tail, lanes=lanes)
    torch.cuda.synchronize()
    print(n, h, w, form, "done", flush=True)
    assert torch.equal(gy, y), int((gy != y).sum())
    assert torch.equal(gb, b) if middle else (gb == 99).all()
    assert torch.equal(gz, z) if third else (gz == 99).all()


PIXELS = {1: 32, 2: 64, 3: 96, 4: 112}


def fits(tile, w):
    """Whether the tile and its patch fit the chip's LDS: the library's own rule"""
    return ((PIXELS[tile] + 2 * w + 3) * 17 + 63) // 64 * 1024 + PIXELS[tile] * 1040 + 6144 <= 160 * 1024


@pytest.fixture(params=[1, 2, 3, 4], ids=lambda t: "tiles%d" % PIXELS[t])
def tile(request):
    from paper_2006_11735_amd import binding as B
    B.icnn_set_tuning("tri_tile", request.param)
    yield request.param
    B.icnn_set_tuning("reset")


# tiles within an image, over several images and ending with the tensor; one pixel; narrow and wide images; more tiles than workgroups at once
@pytest.mark.parametrize("shape", [(2, 14, 14), (1, 1, 1), (1, 7, 7), (2, 9, 30), (1, 23, 17), (1, 1, 40), (1, 40, 1), (3, 16, 8), (16, 2, 7), (7, 2, 8)],
                         ids=lambda s: "x".join(map(str, s)))
def test_equals_the_layers(shape, tile):
    if not fits(tile, shape[2]):
        pytest.skip("the patch does not fit")
    check(*shape)


def test_more_tiles_than_workgroups(tile):
    n = 260 * PIXELS[tile] // 196 + 1
    check(n, 14, 14)
    check(n * 4, 7, 7, third=False)


@pytest.fixture
def smallest_tile():
    from paper_2006_11735_amd import binding as B
    B.icnn_set_tuning("tri_tile", 1)
    yield
    B.icnn_set_tuning("reset")


# workgroups that begin at different taps, one to all nine of them and more (the last block has no next layer: what it fetches ahead is its own next
# tile's first taps)
@pytest.mark.parametrize("tiles", [1, 8, 9, 72, 73, 255, 257, 300])
def test_where_the_weights_begin(tiles, tile):
    check(1, tiles * PIXELS[tile] // 16, 16)
    if tiles > 255:
        check(1, tiles * PIXELS[tile] // 16, 16, third=False)


def test_the_widest_image(smallest_tile):
    from paper_2006_11735_amd import binding as B
    assert fits(1, 210) and not fits(1, 211)
    check(1, 3, 210)
    for forced in (True, False):
        if not forced:
            B.icnn_set_tuning("reset")
        with pytest.raises(B.IcnnError) as e:
            check(1, 3, 211)
        assert e.value.code == B.ICNN_E_UNSUPPORTED


@pytest.mark.parametrize("form", ["hi", "wide", "pc", "pc_mixed"])
def test_requantisation_forms(form, tile):
    check(2, 14, 14, form)
    check(1, 11, 9, form, skip=False)


def test_without_the_third_layer_or_the_middle_output(tile):
    check(2, 14, 14, third=False)
    check(2, 14, 14, middle=False)
    check(30, 3, 3, third=False, middle=False)
    check(1, 11, 9, "pc", third=False)


def test_skip_operand_pitches_and_in_place(tile):
    check(2, 14, 14, skip=False)
    check(2, 14, 14, pitches=(32, 64, 16))
    check(2, 14, 14, in_place=True)


# the skip operand's rescale as one product's high word: the ends of its range, ties at every shift, pairs that reduce to it, pairs it does not take
@pytest.mark.parametrize("rescale", [(1, 0), (30000, 0), (1, 1), (3, 1), (32767, 4), (8000000, 8), (129, 8), (1, 8), (20000 << 4, 10), (20001, 9), (6000000, 30)], ids=str)
def test_skip_rescales(rescale, smallest_tile):
    check(1, 14, 14, rescale=rescale)


def test_the_librarys_choice_of_tiles():
    for n in (6, 48, 84, 128):                       # six: the first that is not taken apart
        check(n, 14, 14)
        check(n, 14, 14, lanes=2)


# below 1176 pixels the library takes the layers apart where each finds in memory what it reads: t2 is stored, at c2's offset 0 and with the pitch that c3
# reads, y likewise for c1, and y is not res.  Every other call is one launch, and in_c_stride of c3 and c1 means nothing there.
@pytest.mark.parametrize("shape", [(1, 25, 47), (1, 24, 49), (6, 14, 14), (1, 7, 7)], ids=lambda s: "x".join(map(str, s)))
def test_on_both_sides_of_the_bound(shape):
    against_oracle(*shape)
    against_oracle(*shape, lanes=2, third=False)


@pytest.mark.parametrize("how", [dict(), dict(pitches=(32, 64, 16)), dict(in_pitch3=272), dict(in_pitch1=1056), dict(offset2=32), dict(offset3=64, third=False),
                                 dict(offset3=64), dict(in_place=True), dict(in_place=True, third=False), dict(middle=False), dict(skip=False),
                                 dict(third=False, in_pitch3=512), dict(middle=False, in_pitch3=272, in_pitch1=1040)], ids=str)
def test_what_a_small_call_needs_to_be_taken_apart(how):
    against_oracle(2, 9, 11, **how)


def against_oracle(n, h, w, skip=True, third=True, middle=True, pitches=(0, 0, 0), in_pitch3=None, in_pitch1=None, offset2=0, offset3=0, in_place=False, lanes=1):
    """pitches: beyond what the channels and their offset take; in_pitch3, in_pitch1: in_c_stride of c3 and c1 (default: what is stored)"""
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng([n, h, w, lanes])
    mid, wide = 256, 1024
    stored = [mid + offset2 + pitches[0], wide + offset3 + pitches[1], mid + pitches[2]]
    l2 = Layer(g, n, h, w, mid, mid, 3, pitch=stored[0])
    l3 = Layer(g, n, h, w, mid, wide, skip=skip, pitch=stored[1], in_pitch=in_pitch3 or stored[0])
    l1 = Layer(g, n, h, w, wide, mid, pitch=stored[2], in_pitch=in_pitch1 or stored[1])
    l2.d.out_c_offset, l3.d.out_c_offset = offset2, offset3
    t = g.integers(0, 128, size=(n, h, w, mid), dtype=np.uint8)
    res = g.integers(0, 256, size=(n, h, w, wide), dtype=np.uint8) if skip else None
    b = l2.oracle(t)
    y = l3.oracle(b, res)
    z = l1.oracle(y)
    gb, gy, gz = (torch.full((n, h, w, c), 99, dtype=torch.uint8, device="cuda:0") for c in stored)
    gres = dev(res) if skip else None
    if in_place:
        assert stored[1] == wide
        gy = gres
    tail = (l1.d, l1.wp, l1.bias, gz) if third else (None,) * 4
    B.iconv2d_triple_brelu(l2.d, dev(t), l2.wp, l2.bias, gb if middle else None, l3.d, l3.wp, l3.bias, gres, gy, *tail, lanes=lanes)
    torch.cuda.synchronize()
    for got, want, at, written in ((gb, b, offset2, middle), (gy, y, offset3, True), (gz, z, 0, third)):
        whole = np.full(got.shape, 99, dtype=np.uint8)
        if written:
            whole[..., at:at + want.shape[3]] = want
        assert (got.cpu().numpy() == whole).all()
    assert len(np.unique(y)) > 3 and len(np.unique(z)) > 3


def test_refused_calls_launch_nothing():
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng(0)
    l2, l3, l1 = Layer(g, 1, 8, 8, 256, 256, 3), Layer(g, 1, 8, 8, 256, 1024, skip=True), Layer(g, 1, 8, 8, 1024, 256)
    t, res = picture(g, 1, 8, 8, 256), picture(g, 1, 8, 8, 1024)
    b, y, z = (torch.full((1, 8, 8, c), 7, dtype=torch.uint8, device="cuda:0") for c in (256, 1024, 256))

    def code(b=b, y=y, z=z, **over):
        d = {"l2": l2.d, "l3": l3.d, "l1": l1.d}
        for k, v in over.items():
            which, field = k.split("__")
            d[which] = B.conv_desc(**{f: getattr(d[which], f) for f, _ in d[which]._fields_})
            setattr(d[which], field, v)
        with pytest.raises(B.IcnnError) as e:
            B.iconv2d_triple_brelu(d["l2"], t, l2.wp, l2.bias, b, d["l3"], l3.wp, l3.bias, res, y, d["l1"], l1.wp, l1.bias, z)
        return e.value.code
    assert code(b=t) == code(y=t) == code(z=t) == code(z=b) == code(z=res) == code(b=res) == B.ICNN_E_UNSUPPORTED
    for over in (dict(l2__bound_q=255), dict(l3__bound_q=255), dict(l3__res_dtype=B.ICNN_S8), dict(l3__res_mode=B.ICNN_RES_POST),
                 dict(l2__in_signed=B.ICNN_IN_U8_FULL), dict(l1__out_mode=B.ICNN_OUT_RAW_S32), dict(l2__stride_h=2, l2__stride_w=2)):
        assert code(**over) == B.ICNN_E_UNSUPPORTED, over
    assert code(l3__h=4) == B.ICNN_E_SHAPE
    torch.cuda.synchronize()
    assert (b == 7).all() and (y == 7).all() and (z == 7).all()
