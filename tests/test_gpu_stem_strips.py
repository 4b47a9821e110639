"""GPU parity of the first layer with its pool where a wave's strip ends in odd places: one to several pooled rows a strip with a shorter
last one, pooled widths around a strip's 14 columns, convolutions of odd height, one and two waves to a strip, pictures a pixel wide, all
requantisation forms, against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu


def run(seed, n, h, w, cin, cout, kh, kw, pad, form="hi", tall=None):
    """form: "hi" one product's high word, "wide" the general form, "pc" per channel.  tall: pad_h, the rows beyond `pad` as rows of zeros."""
    from gpu_util import dev
    from paper_2006_11735_amd import binding as B
    g = np.random.default_rng(seed)
    raw = tall is None and seed % 2 == 0
    x = g.integers(0, 256 if raw else 128, size=(n, h, w, cin), dtype=np.uint8)
    wt = g.integers(-127, 128, size=(cout, kh, kw, cin), dtype=np.int8)
    b = g.integers(-30000, 30001, size=cout).astype(np.int32)
    mul, shift = {"hi": (20000, 24), "wide": (20000 << 14, 38), "pc": (20000, 24)}[form]
    pc = dict(mul_c=g.integers(10000, 30000, size=cout).astype(np.int32), shift_c=g.integers(23, 26, size=cout).astype(np.int32)) if form == "pc" else {}
    xo = x if tall is None else np.pad(x, ((0, 0), (tall - pad, tall - pad), (0, 0), (0, 0)))
    want = O.maxpool2d(O.conv2d(xo, wt, b, stride=2, pad=pad, in_sub128=raw, mul=mul, shift=shift, bound_q=127, **pc), 3, 2, 1)
    d = B.conv_desc(n=n, h=h, w=w, cin=cin, in_c_stride=cin, in_sub128=int(raw), cout=cout, kh=kh, kw=kw, stride_h=2, stride_w=2,
                    pad_h=pad if tall is None else tall, pad_w=pad, out_c_stride=cout, mul=mul, shift=shift, bound_q=127)
    wp = torch.zeros(B.iconv2d_packed_weight_bytes(d), dtype=torch.uint8, device="cuda:0")
    B.iconv2d_prepack_weights(d, dev(wt), wp)
    y = torch.full(want.shape, 99, dtype=torch.uint8, device="cuda:0")
    if form == "pc":
        m, s = dev(pc["mul_c"]), dev(pc["shift_c"])
        packed = torch.zeros(B.iconv2d_packed_channel_params_bytes(d), dtype=torch.uint8, device="cuda:0")
        B.iconv2d_prepack_channel_params(d, B.channel_params(m.data_ptr(), s.data_ptr(), None, None), packed)
        B.iconv2d_maxpool_brelu_pc(d, 3, 2, 1, dev(x), wp, dev(b), packed, y)
    else:
        B.iconv2d_maxpool_brelu(d, 3, 2, 1, dev(x), wp, dev(b), y)
    torch.cuda.synchronize()
    assert (y.cpu().numpy() == want).all()
    assert want.max() > 0


@pytest.mark.parametrize("form", ["hi", "wide", "pc"])
@pytest.mark.parametrize("shape", [
    (1, 30, 56, 3, 64, 7, 7, 3),         # two waves to a strip, exactly a strip wide
    (2, 33, 58, 3, 64, 7, 7, 3),         # a column more; an odd convolution's last row
    (3, 23, 53, 2, 32, 6, 8, 2),
    (40, 41, 57, 3, 64, 7, 7, 3),        # a wave to a strip
    (330, 34, 20, 3, 64, 7, 7, 3),       # two pooled rows a strip, nine in all
    (1000, 26, 20, 3, 32, 7, 7, 3),      # four, seven in all
    (700, 27, 9, 4, 64, 8, 5, 2),
], ids=lambda s: "x".join(map(str, s)))
def test_strips(shape, form):
    run(sum(shape), *shape, form=form)


@pytest.mark.parametrize("shape", [(4, 3, 1, 1, 32, 5, 5, 2), (2, 5, 1, 3, 64, 7, 7, 3), (1, 1, 2, 3, 64, 1, 5, 2), (3, 2, 3, 2, 64, 3, 7, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_pictures_a_pixel_or_two_wide(shape):
    # rows of one to nine bytes: the tensor's first dword holds several of them
    run(sum(shape) * 2, *shape)
    run(sum(shape) * 2 + 1, *shape)


def test_padding_beyond_16_bits():
    run(5, 1, 6, 5, 3, 32, 5, 5, 2, tall=65540)
